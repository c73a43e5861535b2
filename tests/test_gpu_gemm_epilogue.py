"""The GEMM epilogue's way through LDS: every tile shape with ragged rows and
columns, outputs whose rows are 16-byte aligned and not, int32 and fp32 outputs
alone and together, against the exact product of the codes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2411_10948_amd import shiftquant
    shiftquant.load()
    return shiftquant


SHAPES = [  # M, C_out (a multiple of 64: the direct-load kernel), C_in
    (1, 64, 1), (70, 64, 33), (130, 192, 131), (257, 128, 66), (60, 256, 200), (2900, 1024, 2891), (16300, 1024, 764),
    (16384, 768, 3070),
]


def _out(torch, rows, cols, pad, dtype):
    buf = torch.full((rows + 1, cols + pad), -7, dtype=dtype, device="cuda")
    return buf, buf[:rows, :cols]


@pytest.mark.parametrize("M,C_out,C_in", SHAPES)
@pytest.mark.parametrize("pad", [0, 1, 4])
def test_epilogue_edges(sq, M, C_out, C_in, pad):
    import torch
    print(f"epilogue M={M} C_out={C_out} C_in={C_in} pad={pad}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + C_in + pad)
    dY = torch.randn(M, C_out, generator=g, device="cuda") * torch.exp2(-4 * torch.rand(C_out, generator=g, device="cuda"))
    W = torch.randn(C_out, C_in, generator=g, device="cuda")
    c = sq.quantize_grad(dY, 4, 4)
    wq_t, ws = sq.quantize_tensor(W, 8)
    shifted = c.codes().double() * torch.exp2(3.0 - c.group.double())
    ref = (shifted @ wq_t[:, :C_out].t().double()).to(torch.int32)
    alpha = (c.scale[2] * ws[2]) * 0.125
    work = torch.empty(256, dtype=torch.uint8, device="cuda")
    for want_acc, want_out in ((True, True), (True, False), (False, True)):
        abuf, acc = _out(torch, M, C_in, pad, torch.int32)
        obuf, out = _out(torch, M, C_in, pad, torch.float32)
        sq.sq_gemm_dgrad(c.q_fold, c.layout, c.group, c.scale, wq_t, ws, M, C_out, C_in, c.params,
                         acc if want_acc else None, out if want_out else None, work)
        torch.cuda.synchronize()
        if want_acc:
            assert torch.equal(acc, ref)
        if want_out:
            assert torch.equal(out, ref.float() * alpha)
        for buf, on in ((abuf, want_acc), (obuf, want_out)):   # nothing past the output's rows and columns
            assert bool((buf[:M, C_in:] == -7).all()) and bool((buf[M] == -7).all())
            assert on or bool((buf == -7).all())
