"""Products whose inner dimension is not a multiple of the 64-byte K tile, on
every tile shape, with and without appended fold windows and with K split: the
last tile's bytes past K (row padding, poisoned here) must not count.  Against
the exact product of the codes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2411_10948_amd import shiftquant
    shiftquant.load()
    return shiftquant


def _codes(sq, M, C, bits, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(M, C, generator=g, device="cuda") * torch.exp2(-6 * torch.rand(C, generator=g, device="cuda"))
    return sq.quantize_grad(x, bits, 4), g


@pytest.mark.parametrize("M,C_out,C_in", [
    (70, 1, 40), (130, 15, 130), (64, 17, 300), (200, 63, 64), (129, 65, 257), (256, 1000, 200), (2900, 1025, 2900),
    (16300, 1100, 760), (300, 127, 70),
])
@pytest.mark.parametrize("bits", [4, 8])
def test_dgrad_k_tail(sq, M, C_out, C_in, bits):
    import torch
    print(f"dgrad tail M={M} C_out={C_out} C_in={C_in} b={bits}", flush=True)
    c, g = _codes(sq, M, C_out, bits, M + C_out)
    wq_t, ws = sq.quantize_tensor(torch.randn(C_out, C_in, generator=g, device="cuda"), 8)
    ref = ((c.codes().double() * torch.exp2(3.0 - c.group.double())) @ wq_t[:, :C_out].t().double()).to(torch.int32)
    base = (C_out + 63) // 64 * 64
    c.q_fold[:, C_out:base] = 77     # never written by the quantizer
    wq_t.as_strided((C_in, wq_t.stride(0)), (wq_t.stride(0), 1))[:, C_out:] = -55
    acc, _ = sq.gemm_dgrad(c, wq_t, ws, want_acc=True, want_out=False)
    torch.cuda.synchronize()
    assert torch.equal(acc, ref)


@pytest.mark.parametrize("M,C_out,C_in", [(1, 70, 40), (33, 64, 130), (1999, 48, 200), (3152, 768, 768),
                                          (16333, 3072, 768), (1100, 2900, 2900), (5001, 200, 64)])
def test_wgrad_k_tail(sq, M, C_out, C_in):
    import torch
    print(f"wgrad tail M={M} C_out={C_out} C_in={C_in}", flush=True)
    c, g = _codes(sq, M, C_out, 6, M + C_in)
    xq_t, xs = sq.quantize_tensor(torch.randn(M, C_in, generator=g, device="cuda"), 8)
    ref = (c.codes().t().double() @ xq_t[:, :M].t().double()).to(torch.int32)
    for t, v in ((c.q_t, 77), (xq_t, -55)):
        t.as_strided((t.shape[0], t.stride(0)), (t.stride(0), 1))[:, M:] = v
    acc, _ = sq.gemm_wgrad(c, xq_t, xs, want_acc=True, want_out=False)
    torch.cuda.synchronize()
    assert torch.equal(acc, ref)
