"""Every tile shape and K split that the GEMM's plan picks, with ragged rows,
columns and inner dimensions and with appended fold windows: both backward
products of a layer against the exact products of its codes."""
import pytest

from tests.gemm_plan import gemm_plan

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
    (8192, 2100, 4096),     # 256 x 256; 128 x 384
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


# many rows, short inner dimensions: dX tile of row-major codes (0: the
# register-staged kernel) without and with appended fold windows
STAGED, WIDE = (0, 0), (256, 128)
NARROW = [
    (32767, 16, 16, (64, 128), (64, 128)),
    (32768, 10, 8, STAGED, STAGED),
    (33001, 128, 32, STAGED, STAGED),
    (33001, 64, 48, STAGED, STAGED),
    (262145, 30, 96, STAGED, STAGED),
    (262145, 64, 100, STAGED, WIDE),
    (262145, 64, 97, WIDE, WIDE),             # rows that are not 16-byte aligned
    (70001, 48, 132, STAGED, STAGED),
    (70001, 64, 129, (64, 128), (64, 128)),
    (33001, 64, 30, (256, 64), (256, 64)),
    (33001, 64, 13, STAGED, STAGED),
    (190001, 17, 300, STAGED, WIDE),
    (40001, 129, 32, (256, 64), (256, 64)),
    (33333, 65, 48, (256, 64), (256, 64)),
    (32769, 200, 64, (256, 64), (256, 64)),
    (262145, 96, 49, (64, 64), (64, 64)),
    (70001, 128, 65, WIDE, WIDE),
    (65281, 100, 128, WIDE, WIDE),
    (190001, 65, 300, WIDE, WIDE),
]


@pytest.mark.parametrize("M,C_out,C_in,tile,tile_ext", NARROW)
@pytest.mark.parametrize("bits,tiled", [(4, False), (6, False), (6, True)])
def test_narrow_products(sq, M, C_out, C_in, tile, tile_ext, bits, tiled):
    assert gemm_plan(sq, M, C_in, C_out) == (*tile, 0)
    assert gemm_plan(sq, M, C_in, C_out, ext=True) == (*tile_ext, 0)
    test_every_tile_and_split(sq, M, C_out, C_in, bits, tiled)


# the GEMM-based comparison's products (a K segment per group) on those tiles
@pytest.mark.parametrize("M,C_out,C_in", [(33001, 96, 40), (262145, 70, 61), (70001, 130, 100)])
@pytest.mark.parametrize("bits", [4, 8])
def test_narrow_grouped(sq, M, C_out, C_in, bits):
    import torch
    print(f"narrow grouped M={M} C_out={C_out} C_in={C_in} b={bits}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + C_out + bits)
    dY = torch.randn(M, C_out, generator=g, device="cuda") * torch.exp2(-6 * torch.rand(C_out, generator=g, device="cuda"))
    c = sq.quantize_grad(dY, bits, 4)
    wq_t, ws = sq.quantize_tensor(torch.randn(C_out, C_in, generator=g, device="cuda"), 8)
    A, dX = sq.gemm_dgrad_grouped(c, wq_t, ws, want_acc=True)
    torch.cuda.synchronize()
    ref = ((c.codes().double() * torch.exp2(3.0 - c.group.double())) @ wq_t[:, :C_out].t().double()).to(torch.int32)
    assert torch.equal(A, ref)
    assert torch.equal(dX, ref.float() * (c.scale[2] * ws[2] * 0.125))


# the forward's per-column scales on the register-staged kernel
@pytest.mark.parametrize("M,C_in,C_out", [(33001, 70, 32), (32768, 64, 44)])
@pytest.mark.parametrize("bits", [4, 8])
def test_narrow_forward(sq, M, C_in, C_out, bits):
    import torch
    print(f"narrow forward M={M} C_in={C_in} C_out={C_out} b={bits}", flush=True)
    assert gemm_plan(sq, M, C_out, C_in) == (0, 0, 0)
    g = torch.Generator(device="cuda").manual_seed(M + C_out + bits)
    x = torch.randn(M, C_in, generator=g, device="cuda") * torch.exp2(-6 * torch.rand(C_in, generator=g, device="cuda"))
    c = sq.quantize_grad(x, bits, 4)
    wq, ws = sq.quantize_channels(torch.randn(C_out, C_in, generator=g, device="cuda"), 8)
    A, Y = sq.gemm_forward(c, wq, ws, want_acc=True)
    torch.cuda.synchronize()
    ref = ((c.codes().double() * torch.exp2(3.0 - c.group.double())) @ wq[:, :C_in].t().double()).to(torch.int32)
    assert torch.equal(A, ref)
    assert torch.equal(Y, ref.float() * ((c.scale[2] * ws[:, 2]) * 0.125)[None, :])


# 256 x 256 tiles with every dimension ragged, and products that take two
# launches, the rows of whole rounds of large tiles and the rest: plan of dX, dW
LARGE = [
    (10976, 3394, 1025, (256, 256, 0), (128, 128, 0)),
    (3332, 3488, 3658, (256, 256, 0), (256, 256, 0)),
    (4386, 1538, 4048, (128, 128, 4096), (128, 128, 0)),
    (1565, 9733, 1748, (128, 128, 0), (128, 128, 9216)),
    (3233, 3131, 5768, (128, 384, 2816), (128, 384, 2816)),
]


@pytest.mark.parametrize("M,C_out,C_in,plan_dx,plan_dw", LARGE)
@pytest.mark.parametrize("bits,tiled", [(4, False), (6, True), (8, False)])
def test_large_tiles_and_row_splits(sq, M, C_out, C_in, plan_dx, plan_dw, bits, tiled):
    assert gemm_plan(sq, M, C_in, C_out) == plan_dx
    assert gemm_plan(sq, C_out, C_in, M) == plan_dw
    assert sq.sq_gemm_wgrad_workspace_size(M, C_out, C_in, sq.Params.make(bits)) == 0   # K not split
    test_every_tile_and_split(sq, M, C_out, C_in, bits, tiled)


# code matrices of 2^31 bytes and more (long rows), past the pipelined kernel's
# offsets: the register-staged kernel's two tiles, with fold windows, K split
# and the ranged product's separate maxima
@pytest.mark.parametrize("M,C_out,C_in,bits,ld_fold,ld_t", [
    (130, 40, 200, 8, 1 << 24, 1 << 26),
    (3332, 3488, 3658, 4, 655360, 655360),
    (20001, 130, 72, 6, 114688, 1 << 24),
])
def test_operands_past_31_bits(sq, M, C_out, C_in, bits, ld_fold, ld_t):
    import torch
    print(f"past 31 bits M={M} C_out={C_out} C_in={C_in} b={bits}", flush=True)
    assert M * ld_fold >= 1 << 31 and C_out * ld_t >= 1 << 31
    g = torch.Generator(device="cuda").manual_seed(M + bits)
    dY = torch.randn(M, C_out, generator=g, device="cuda") * torch.exp2(-6 * torch.rand(C_out, generator=g, device="cuda"))
    c = sq.quantize_grad(dY, bits, 4)
    wq_t, ws = sq.quantize_tensor(torch.randn(C_out, C_in, generator=g, device="cuda"), 8)
    xq_t, xs = sq.quantize_tensor(torch.randn(M, C_in, generator=g, device="cuda"), 8)

    def far(t, ld):   # the same codes in rows of ld bytes
        out = torch.empty((t.shape[0], ld), dtype=torch.int8, device="cuda")
        out[:, :t.shape[1]] = t
        return out

    q_fold, q_t = c.q_fold, c.q_t
    A0, dX0 = sq.gemm_dgrad(c, wq_t, ws, want_acc=True)
    B0, dW0 = sq.gemm_wgrad(c, xq_t, xs, want_acc=True)
    c.q_fold = far(q_fold, ld_fold)
    A, dX = sq.gemm_dgrad(c, wq_t, ws, want_acc=True)
    ranges = torch.empty(sq.sq_gemm_dgrad_range_slabs(M), C_in, dtype=torch.int32, device="cuda")
    dX_r = torch.empty_like(dX)
    w = torch.empty(max(256, sq.sq_gemm_dgrad_workspace_size(M, C_out, C_in, c.params)), dtype=torch.uint8, device="cuda")
    sq.sq_gemm_dgrad_ranged(c.q_fold, c.layout, c.group, c.scale, wq_t, ws, M, C_out, C_in, c.params, None, dX_r, ranges, w)
    c.q_fold, c.q_t = q_fold, far(q_t, ld_t)
    B, dW = sq.gemm_wgrad(c, xq_t, xs, want_acc=True)
    torch.cuda.synchronize()
    q = q_t[:, :M].t().double()
    assert torch.equal(A, ((q * torch.exp2(3.0 - c.group.double())) @ wq_t[:, :C_out].t().double()).to(torch.int32))
    assert torch.equal(B, (q.t().contiguous() @ xq_t[:, :M].t().double()).to(torch.int32))
    assert torch.equal(A, A0) and torch.equal(B, B0)
    assert torch.equal(dX, dX0) and torch.equal(dX_r, dX0) and torch.equal(dW, dW0)
    top = torch.zeros(ranges.shape[0] * 32, C_in, device="cuda")
    top[:M] = dX.abs()
    assert torch.equal(ranges.view(torch.float32), top.view(-1, 32, C_in).amax(1))


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
