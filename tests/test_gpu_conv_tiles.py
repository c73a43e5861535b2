"""The conv input gradient of the per-tap kernel, on each of its tile shapes, and
of the staged window, at the edges of their tap masks: windows up to 15 x 15,
one-sided padding, images smaller than the window, rows of several images in one
tile, and all fold cases, against the oracle."""
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


CASES = [  # N, H, W, C_out, C_in, KH, KW, PH, PW, bits
    (3, 2, 2, 70, 65, 3, 3, 1, 1, 4),         # every pixel at a border; 64 x 64 tiles
    (1, 5, 6, 66, 130, 15, 15, 14, 14, 4),    # the largest window, larger than the image
    (2, 9, 4, 100, 64, 1, 15, 0, 7, 6),
    (2, 4, 9, 65, 72, 15, 1, 7, 0, 8),
    (5, 7, 7, 130, 200, 3, 3, 1, 1, 8),       # images of 49 pixels
    (40, 14, 14, 72, 136, 3, 3, 1, 1, 6),     # 64 x 128 tiles
    (64, 20, 20, 66, 136, 3, 3, 0, 2, 4),     # 128 x 128 tiles, unequal padding
    (16, 50, 45, 80, 24, 3, 3, 1, 1, 6),      # a narrow output, 64 x 64 tiles
    (9, 90, 66, 70, 24, 3, 3, 1, 1, 6),       # 256 x 64 tiles
    # the staged window: its widest rows, images smaller than a tile with several
    # fold windows, 9 taps in a row, every dimension ragged
    (12, 90, 62, 70, 33, 3, 3, 1, 1, 4),
    (4099, 4, 4, 129, 20, 3, 3, 1, 1, 8),
    (260, 16, 16, 65, 64, 1, 9, 0, 4, 6),
    (20, 62, 55, 64, 63, 1, 7, 0, 3, 8),
]


@pytest.mark.parametrize("N,H,W,C_out,C_in,KH,KW,PH,PW,bits", CASES)
def test_conv_dgrad_tiles(sq, N, H, W, C_out, C_in, KH, KW, PH, PW, bits):
    import torch
    print(f"conv tiles N={N} {H}x{W} {C_out}->{C_in} {KH}x{KW} P={PH},{PW} b={bits}", flush=True)
    rng = np.random.default_rng(N * 100 + H + C_in)
    Ho, Wo = H + 2 * PH - KH + 1, W + 2 * PW - KW + 1
    dY = (rng.standard_normal((N * Ho * Wo, C_out)) * 2.0 ** -rng.uniform(0, 6, C_out)).astype(np.float32)
    Wt = (rng.standard_normal((C_out, KH * KW * C_in)) * 0.05).astype(np.float32)
    c = sq.quantize_grad(_dev(dY), bits, 4)
    wq_t, ws = sq.quantize_tensor(_dev(Wt), 8)
    acc, dX = sq.conv_dgrad(c, wq_t, ws, N, H, W, KH, KW, PH, PW, want_acc=True)
    torch.cuda.synchronize()
    q, g, gs, _ = oracle.quantize_grad(dY, bits, 4)
    wq, wsr = oracle.quantize_tensor(Wt, 8)
    A = oracle.conv_dgrad(q, g, 4, wq, N, H, W, KH, KW, PH, PW)
    assert np.array_equal(acc.cpu().numpy(), A)
    np.testing.assert_array_equal(dX.cpu().numpy(), oracle.dequant_dgrad(A, gs["d0"], wsr["d0"], 4))
