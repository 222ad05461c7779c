"""Histograms of walkers that weights hold on one level: every visit of a
workgroup then counts on one word in LDS, the most that its 16-bit counts at
L = 128 can take between two flushes, within a sweep and from one sweep to the
next."""
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


# the smallest walker number with four waves in every workgroup, and one wave;
# the ground state (an even level) and two neighbours turned over (an odd one)
@pytest.mark.parametrize("L,W", [(128, 12289), (128, 40), (96, 12289)])
@pytest.mark.parametrize("level", [0, 3])
@pytest.mark.parametrize("nsweeps", [2, 5])
def test_held_on_one_level(ctx, L, W, level, nsweeps):
    N, K, seed = L * L, L * L // 2, 19
    one = np.ones(N, dtype=np.int8)
    if level == 3:
        one[[5 * L + 7, 5 * L + 8]] = -1
    spins = torch.from_numpy(one).cuda().repeat(W, 1).contiguous()
    E = torch.full((W,), 4 * level - 2 * N, dtype=torch.int64, device="cuda")
    # accepted by r32 = 0 alone, which no draw of this seed is (12289 walkers, five sweeps)
    lnW = -1000.0 * np.abs(np.arange(K + 1) - level)
    H = torch.zeros(K + 1, dtype=torch.int64, device="cuda")
    ctx.muca_sweeps(L, spins, E, lnW, seed, 0, nsweeps, True, H=H)
    torch.cuda.synchronize()
    want = np.zeros(K + 1, dtype=np.int64)
    want[level] = W * N * nsweeps
    assert np.array_equal(H.cpu().numpy(), want)
    assert torch.equal(spins, torch.from_numpy(one).cuda().expand(W, N))
    assert bool((E == 4 * level - 2 * N).all())
    # the oracle's walkers stay there too (a few of them: they are independent)
    s, e = np.tile(one, 3), np.full(3, 4 * level - 2 * N, dtype=np.int64)
    h = oracle.muca_sweeps(L, s, e, lnW, seed, 0, nsweeps, True)
    assert h[level] == h.sum() == 3 * N * nsweeps
