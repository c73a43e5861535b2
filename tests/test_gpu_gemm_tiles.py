"""Every tile shape and K split that the GEMM's plan picks, with ragged rows,
columns and inner dimensions and with appended fold windows: both backward
products of a layer against the exact products of its codes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2411_10948_amd import shiftquant
    shiftquant.load()
    return shiftquant


LAYERS = [  # M, C_out, C_in: tile of dX; tile and splits of dW
    (8200, 1100, 4096),     # 128 x 192; 128 x 192
    (8192, 2100, 4096),     # 256 x 128; 128 x 384
    (16384, 3072, 768),     # 128 x 384; 128 x 384 in 5
    (12544, 256, 1024),     # 256 x 128; 64 x 64 in 8
    (16000, 780, 770),      # 256 x 128; 128 x 128 in 5
    (4096, 2048, 2048),     # 128 x 128; 128 x 128
    (2000, 500, 300),       # 64 x 128; 64 x 64
    (9000, 200, 1025),      # 64 x 128; 64 x 128 in 12
    (100, 3000, 2100),      # 64 x 64; 128 x 128
    (257, 100, 200),        # 64 x 128; 64 x 128
    (3000, 768, 768),       # 64 x 128; 64 x 64
]


@pytest.mark.parametrize("M,C_out,C_in", LAYERS)
@pytest.mark.parametrize("bits,tiled", [(4, False), (6, True), (8, False)])
def test_every_tile_and_split(sq, M, C_out, C_in, bits, tiled):
    import torch
    print(f"tiles M={M} C_out={C_out} C_in={C_in} b={bits} tiled={tiled}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + C_out + bits)
    dY = torch.randn(M, C_out, generator=g, device="cuda") * torch.exp2(-6 * torch.rand(C_out, generator=g, device="cuda"))
    c = sq.quantize_grad(dY, bits, 4, tiled=tiled)
    wq_t, ws = sq.quantize_tensor(torch.randn(C_out, C_in, generator=g, device="cuda"), 8, tiled=tiled)
    xq_t, xs = sq.quantize_tensor(torch.randn(M, C_in, generator=g, device="cuda"), 8, tiled=tiled)
    A, dX = sq.gemm_dgrad(c, wq_t, ws, want_acc=True)
    B, dW = sq.gemm_wgrad(c, xq_t, xs, want_acc=True)
    torch.cuda.synchronize()
    rows = sq.untile if tiled else (lambda t: t)
    q = c.codes().double()
    ref = ((q * torch.exp2(3.0 - c.group.double())) @ rows(wq_t)[:, :C_out].t().double()).to(torch.int32)
    assert torch.equal(A, ref)
    assert torch.equal(dX, ref.float() * (c.scale[2] * ws[2] * 0.125))
    ref = (q.t().contiguous() @ rows(xq_t)[:, :M].t().double()).to(torch.int32)
    assert torch.equal(B, ref)
    assert torch.equal(dW, ref.float() * ((c.scale[2] * xs[2]) * torch.exp2(-c.group.float()))[:, None])
