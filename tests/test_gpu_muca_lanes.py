"""Multicanonical sweeps without counting on both sides of the walker numbers
from which one lane per walker is taken, bit for bit against the oracle, with an
unfilled last wave and a threshold of 2^32 - 1 besides; and tables with that
threshold counted, for every row shape."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
mcs = pytest.importorskip("paper_1709_04394_amd")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return mcs.Context(0)


@pytest.mark.parametrize("L,W", [(4, 32768), (4, 32769), (4, 200001), (8, 65536), (8, 65537), (12, 90112), (12, 90113),
                                 (12, 294912), (12, 294913), (16, 106496), (16, 106497)])
@pytest.mark.parametrize("step", [None, 3e-10])
def test_walker_numbers(ctx, L, W, step):
    k = np.arange(L * L // 2 + 1)
    lnW = -0.35 * (4.0 * k - 2.0 * L * L) if step is None else -step * k
    spins, E = ctx.muca_start(L, W, 41)
    ctx.muca_sweeps(L, spins, E, lnW, 41, (1 << 32) - 1, 2, False)
    torch.cuda.synchronize()
    os_, oE = oracle.muca_start(L, W, 41, 0)
    oracle.muca_sweeps(L, os_, oE, lnW, 41, (1 << 32) - 1, 2, False)
    assert np.array_equal(E.cpu().numpy(), oE)
    assert np.array_equal(spins.cpu().numpy().reshape(-1), os_)


@pytest.mark.parametrize("L,W", [(4, 33), (8, 4113), (12, 33), (16, 33), (24, 33), (32, 33), (48, 33), (64, 33), (96, 17),
                                 (128, 17)])
def test_threshold_next_to_one_counted(ctx, L, W):
    # flat weights but for thresholds of 2^32 - 1 downwards: the walkers press
    # against the window's end
    K = L * L // 2
    lnW = -3e-10 * (K - np.arange(K + 1))
    spins, E = ctx.muca_start(L, W, 43)
    H = torch.zeros(K + 1, dtype=torch.int64, device="cuda")
    ctx.muca_sweeps(L, spins, E, lnW, 43, 5, 3, True, H=H)
    torch.cuda.synchronize()
    os_, oE = oracle.muca_start(L, W, 43, 0)
    oH = oracle.muca_sweeps(L, os_, oE, lnW, 43, 5, 3, True)
    assert oH[K] > 0
    assert np.array_equal(H.cpu().numpy(), oH)
    assert np.array_equal(E.cpu().numpy(), oE)
    assert np.array_equal(spins.cpu().numpy().reshape(-1), os_)
