"""The gradient quantizer's finalize (k_final_groups, k_final_place) at the
edges of its 64-channel groups and 256-channel blocks, with one and with
several fold windows, from the quantizer's own abs-max pass and from the
producer's ranges: codes, groups, scale and every word of the fold layout
against the oracle, bit for bit."""
import numpy as np
import pytest

from tests.test_gpu_parity import _dev, check_quant

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2411_10948_amd import shiftquant
    shiftquant.load()
    return shiftquant


@pytest.mark.parametrize("bits,ng", [(4, 4), (6, 4), (8, 8), (2, 8)])
@pytest.mark.parametrize("C", [1, 7, 64, 65, 255, 257, 704, 1025])
def test_finalize_group_edges(sq, C, bits, ng):
    import torch
    print(f"finalize C={C} b={bits} ng={ng}", flush=True)
    rng = np.random.default_rng(1000 * C + 10 * bits + ng)
    M = 203
    # channel ranges over 2^-9 .. 1, so every group and window has channels
    dY = (rng.uniform(-1, 1, (M, C)) * 2.0 ** -rng.uniform(0, 9, C)).astype(np.float32)
    a = sq.quantize_grad(_dev(dY), bits, ng)
    bits_dY = np.abs(dY).view(np.uint32)
    ranges = np.stack([bits_dY[i:i + 32].max(axis=0) for i in range(0, M, 32)])
    b = sq.quantize_grad_from_ranges(_dev(dY), torch.from_numpy(ranges.view(np.int32)).cuda(), bits, ng)
    torch.cuda.synchronize()
    check_quant(sq, a, dY, bits, ng, 0, 0, 0)
    for name in ("q_fold", "q_t", "group", "layout", "scale"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name


# channel counts whose shift counts take more than one batch of loads (above
# 16384) and, from 32705 in at most 8 slabs, a wave per 64 channels; many slabs
# (here a range per row: a part of them per block where the scratch holds the
# parts) on both sides of the direct path's limits (512 slabs, 16384 ranges)
@pytest.mark.parametrize("M,C", [(9, 16385), (8, 32704), (8, 32705), (9, 40000), (5, 70001),
                                 (512, 1), (513, 1), (700, 3), (6000, 64), (128, 128), (129, 128), (3001, 130), (2000, 1025)])
@pytest.mark.parametrize("bits,ng", [(4, 4), (6, 4)])
def test_finalize_many_channels_or_slabs(sq, M, C, bits, ng):
    import torch
    print(f"finalize M={M} C={C} b={bits}", flush=True)
    rng = np.random.default_rng(M + C + bits)
    dY = (rng.uniform(-1, 1, (M, C)) * 2.0 ** -rng.uniform(0, 9, C)).astype(np.float32)
    d = _dev(dY)
    a = sq.quantize_grad(d, bits, ng)
    b = sq.quantize_grad_from_ranges(d, d.abs().view(torch.int32).contiguous(), bits, ng)
    torch.cuda.synchronize()
    check_quant(sq, a, dY, bits, ng, 0, 0, 0)
    for name in ("q_fold", "q_t", "group", "layout", "scale"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
