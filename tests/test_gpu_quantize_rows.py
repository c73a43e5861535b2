"""Per-row weight codes (k_quantize_rows): column counts around the 4-column
words and the 64-lane wave, aligned and unaligned rows, rows whose maximum is
zero, tiny or not finite, against the oracle; nothing past a row's codes."""
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


@pytest.mark.parametrize("rows,cols", [(1, 1), (5, 3), (7, 4), (9, 63), (4, 255), (6, 257), (3, 1000), (33, 2051),
                                       (130, 2), (129, 16), (67, 17), (200, 33), (131, 64), (35, 70), (21, 128)])   # several rows per wave
@pytest.mark.parametrize("pad", [0, 1, 4])
def test_quantize_rows_edges(sq, rows, cols, pad):
    import torch
    print(f"rows {rows} x {cols} pad {pad}", flush=True)
    rng = np.random.default_rng(rows * 1000 + cols)
    W = rng.standard_normal((rows, cols)).astype(np.float32)
    W[0] = 0.0
    if rows > 4:
        W[1, cols // 2] = np.inf
        W[2, 0] = np.nan
        W[3] = 1e-30
    buf = torch.full((rows, cols + pad), 3.0e38, dtype=torch.float32, device="cuda")
    buf[:, :cols] = _dev(W)
    q = torch.full((rows, (cols + 15) // 16 * 16 + 16), 99, dtype=torch.int8, device="cuda")
    scales = torch.zeros((rows, 4), dtype=torch.float32, device="cuda")
    sq.sq_quantize_channels(buf[:, :cols], 8, 0, False, q, scales, None)
    torch.cuda.synchronize()
    got, sc = q.cpu().numpy(), scales.cpu().numpy()
    for r in range(rows):
        q_ref, s_ref = oracle.quantize_tensor(W[r:r + 1], 8)
        assert np.array_equal(got[r, :cols], q_ref[0]), r
        assert sc[r, 2] == np.float32(s_ref["d0"]) and sc.view(np.int32)[r, 3] == s_ref["flags"], r
    assert (got[:, cols:] == 99).all()
