"""Producer-side channel ranges from the loss-propagation GEMM (sq_gemm_dgrad_ranged),
anchored on the oracle: dX equals the oracle's dX bit for bit (and
sq_gemm_dgrad's), every 32-row slab maximum equals the maximum of the oracle's
|dX| over those rows (bit patterns), and quantizing dX with those ranges gives
the oracle quantizer's codes, groups and scale on the oracle's dX (and exactly
the quantizer's own abs-max pass).  Inputs are seeded and synthetic."""
import numpy as np
import pytest

import oracle
from tests.gemm_plan import gemm_plan
from tests.test_gpu_parity import _dev, _grad, check_quant

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2411_10948_amd import shiftquant
    shiftquant.load()
    return shiftquant


RANGE_CASES = [  # M, C_out, C_in, bits, N_G
    (1000, 256, 1024, 4, 4),
    (777, 300, 200, 6, 4),      # appended fold windows, ragged M and C
    (40, 128, 96, 4, 4),        # a single row tile
    (4099, 768, 3072, 6, 4),    # the MLP chain's down-projection
    (65, 64, 48, 8, 3),
    (8000, 1024, 1536, 6, 4),   # fold windows
    (8000 - 40, 1024, 1536, 4, 4),   # one window, ragged rows
]


@pytest.mark.parametrize("case", RANGE_CASES, ids=["x".join(map(str, c)) for c in RANGE_CASES])
def test_dgrad_ranges(sq, case):
    import torch
    M, C_out, C_in, bits, ng = case
    print(f"dgrad ranges {case}", flush=True)
    rng = np.random.default_rng(M + C_in)
    dY = _grad(M, C_out, seed=M)
    Wt = (rng.standard_normal((C_out, C_in)) * 0.02).astype(np.float32)
    codes = sq.quantize_grad(_dev(dY), bits, ng)
    wq_t, ws = sq.quantize_tensor(_dev(Wt), 8, transpose=True)
    _, dX0 = sq.gemm_dgrad(codes, wq_t, ws)
    slabs = sq.sq_gemm_dgrad_range_slabs(M)
    assert slabs == (M + 31) // 32
    dX = torch.empty((M, C_in), dtype=torch.float32, device="cuda")
    ranges = torch.full((slabs, C_in), -1, dtype=torch.int32, device="cuda")
    wsz = sq.sq_gemm_dgrad_workspace_size(M, C_out, C_in, codes.params)
    ws_d = torch.empty(max(wsz, 256), dtype=torch.uint8, device="cuda")
    sq.sq_gemm_dgrad_ranged(codes.q_fold, codes.layout, codes.group, codes.scale, wq_t, ws, M, C_out, C_in,
                            codes.params, None, dX, ranges, ws_d)
    torch.cuda.synchronize()
    assert torch.equal(dX, dX0)
    # the oracle's dX of the same layer
    oracle.set_threads(16)
    q_ref, g_ref, s_ref, _ = oracle.quantize_grad(dY, bits, ng)
    wq_ref, ws_ref = oracle.quantize_tensor(Wt, 8)
    dX_ref = oracle.dequant_dgrad(oracle.dgrad(q_ref, g_ref, ng, wq_ref), s_ref["d0"], ws_ref["d0"], ng)
    np.testing.assert_array_equal(dX.cpu().numpy().view(np.uint32), dX_ref.view(np.uint32))
    xb = dX_ref.view(np.uint32) & 0x7FFFFFFF
    pad = slabs * 32 - M
    ref = np.concatenate([xb, np.zeros((pad, C_in), np.uint32)]).reshape(slabs, 32, C_in).max(axis=1)
    np.testing.assert_array_equal(ranges.cpu().numpy().view(np.uint32), ref)
    # the next layer's quantizer fed these ranges
    a = sq.quantize_grad(dX, bits, ng)
    b = sq.quantize_grad_from_ranges(dX, ranges, bits, ng)
    torch.cuda.synchronize()
    check_quant(sq, b, dX_ref, bits, ng, 0, 0, 0)
    for name in ("q_fold", "q_t", "group", "layout"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    assert torch.equal(a.scale, b.scale)


RANGE_TILES = [  # M, C_out, C_in: every tile shape, ragged rows and columns
    (65, 1152, 70, (64, 64)),
    (65, 320, 65, (64, 128)),
    (9890, 320, 537, (128, 128)),
    (5555, 256, 1793, (128, 192)),
    (11207, 704, 657, (128, 384)),
    (9795, 256, 1283, (256, 128)),
    (9830, 3392, 1173, (256, 256)),
    (40001, 192, 61, (256, 64)),
]


# the ranged product runs the tile that its plan prices, with and without fold
# windows: dX as the plain product's, the maxima those of the stored dX
@pytest.mark.parametrize("M,C_out,C_in,tile", RANGE_TILES)
@pytest.mark.parametrize("bits", [4, 8])
def test_dgrad_ranges_every_tile(sq, M, C_out, C_in, tile, bits):
    import torch
    print(f"dgrad ranges tile M={M} C_out={C_out} C_in={C_in} b={bits}", flush=True)
    assert gemm_plan(sq, M, C_in, C_out)[:2] == tile
    g = torch.Generator(device="cuda").manual_seed(M + bits)
    dY = torch.randn(M, C_out, generator=g, device="cuda") * torch.exp2(-6 * torch.rand(C_out, generator=g, device="cuda"))
    c = sq.quantize_grad(dY, bits, 4)
    wq_t, ws = sq.quantize_tensor(torch.randn(C_out, C_in, generator=g, device="cuda"), 8)
    _, ref = sq.gemm_dgrad(c, wq_t, ws)
    slabs = sq.sq_gemm_dgrad_range_slabs(M)
    dX = torch.full((M, C_in), float("nan"), device="cuda")
    ranges = torch.full((slabs + 1, C_in), -1, dtype=torch.int32, device="cuda")
    w = torch.empty(max(256, sq.sq_gemm_dgrad_workspace_size(M, C_out, C_in, c.params)), dtype=torch.uint8, device="cuda")
    sq.sq_gemm_dgrad_ranged(c.q_fold, c.layout, c.group, c.scale, wq_t, ws, M, C_out, C_in, c.params, None, dX, ranges, w)
    torch.cuda.synchronize()
    assert torch.equal(dX, ref)
    top = torch.zeros(slabs * 32, C_in, device="cuda")
    top[:M] = dX.abs()
    assert torch.equal(ranges[:slabs].view(torch.float32), top.view(slabs, 32, C_in).amax(1))
    assert bool((ranges[slabs] == -1).all())
