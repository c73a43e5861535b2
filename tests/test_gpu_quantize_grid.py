"""The quantizers that write transposed codes onto the padded pixel grid
(k_quantize_grid, k_quantize8) at the edges of their tiles: widths around the divisors of
128, the longest single-tile width, several tiles per image row, tiles that
span images, leads of 0 to 7 columns and channel counts around 64.  Every byte
of both grids against the oracle's codes laid out by numpy, and the folded
operand against the one of the plain gradient quantizer."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2411_10948_amd import shiftquant
    shiftquant.load()
    return shiftquant


def _grid(codes, N, Hc, Wc, top, left, Hp, Wp, ld):
    """codes [N*Hc*Wc, C] on the padded grid [C, ld]."""
    C = codes.shape[1]
    full = np.zeros((C, N, Hp, Wp), np.int8)
    full[:, :, top:top + Hc, left:left + Wc] = codes.reshape(N, Hc, Wc, C).transpose(3, 0, 1, 2)
    out = np.zeros((C, ld), np.int8)
    out[:, :N * Hp * Wp] = full.reshape(C, -1)
    return out


CASES = [  # N, H, W, C, KH, KW, PH, PW
    (3, 5, 1, 8, 3, 3, 1, 1), (2, 3, 7, 72, 3, 3, 1, 1), (5, 14, 14, 64, 3, 3, 1, 1), (1, 28, 28, 16, 3, 3, 1, 1),
    (2, 2, 43, 24, 5, 15, 2, 7), (2, 3, 64, 8, 1, 3, 0, 1), (1, 2, 127, 40, 3, 3, 1, 1), (2, 3, 128, 8, 3, 1, 1, 0),
    (1, 3, 129, 64, 3, 3, 1, 1), (2, 2, 126, 8, 3, 5, 1, 2), (1, 2, 257, 136, 3, 3, 1, 1), (1, 1, 300, 8, 1, 7, 0, 3),
    (9, 1, 9, 8, 1, 3, 0, 1),
    # 128 consecutive pixels a tile: rows that whole-row tiles fill badly, and
    # (stochastic) any multiple of 8; tiles of many images; the last tile ragged
    (2, 3, 72, 72, 3, 3, 1, 1), (1, 3, 144, 64, 3, 3, 1, 1), (2, 3, 48, 8, 3, 1, 1, 0), (7, 3, 8, 136, 3, 3, 1, 1),
    (1, 1, 80, 40, 1, 1, 0, 0), (2, 2, 200, 24, 3, 3, 1, 1),
]


@pytest.mark.parametrize("N,H,W,C,KH,KW,PH,PW", CASES)
@pytest.mark.parametrize("bits,mode", [(4, 0), (6, 1)])
def test_quantize_grid_edges(sq, N, H, W, C, KH, KW, PH, PW, bits, mode):
    import torch
    print(f"grid N={N} H={H} W={W} C={C} K={KH}x{KW} P={PH},{PW} b={bits} mode={mode}", flush=True)
    rng = np.random.default_rng(N * 1000 + W * 10 + C + mode)
    Ho, Wo = H + 2 * PH - KH + 1, W + 2 * PW - KW + 1
    Hp, Wp = H + 2 * PH, (W + 2 * PW + 15) // 16 * 16
    dY = (rng.standard_normal((N * Ho * Wo, C)) * 2.0 ** -rng.uniform(0, 6, C)).astype(np.float32)
    X = rng.standard_normal((N * H * W, C)).astype(np.float32)
    p = sq.Params.make(bits, 4, mode, 5, 3)
    plan = sq.ConvBackwardPlan(N, H, W, C, C, KH, KW, PH, PW, p)
    plan.quantize_input(_dev(X))
    plan.quantize(_dev(dY))
    plain = sq.quantize_grad(_dev(dY), bits, 4, mode, 5, 3)
    torch.cuda.synchronize()
    q_ref, g_ref, _, _ = oracle.quantize_grad(dY, bits, 4, mode, 5, 3)
    x_ref, _ = oracle.quantize_tensor(X, 8)
    assert np.array_equal(plan.group.cpu().numpy(), g_ref)
    assert np.array_equal(plan.q_tp.cpu().numpy(), _grid(q_ref, N, Ho, Wo, 0, 0, Hp, Wp, plan.q_tp.shape[1]))
    assert np.array_equal(plan.x_grid.cpu().numpy(), _grid(x_ref, N, H, W, PH, PW, Hp, Wp, plan.x_grid.shape[1]))
    assert torch.equal(plan.q_fold[:, :C], plain.q_fold[:, :C]) and torch.equal(plan.layout, plain.layout)
    ext = int(plan.layout[1])   # appended columns in use: their channels' codes
    used = (plan.layout[32:32 + ext] >= 0).nonzero().flatten() + int(plan.layout[2])
    assert torch.equal(plan.q_fold[:, used], plain.q_fold[:, used])
