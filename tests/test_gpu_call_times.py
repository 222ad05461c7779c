"""Times of calls away from the benchmark's sizes, where a rule that chooses
between kernels can choose the slower one: each against a bound between the
times of the two kernels, well away from both."""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
mcs = pytest.importorskip("paper_1709_04394_amd")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return mcs.Context(0)


def _us(call, n=9):
    """Shortest of n calls, each waited for, after one that is not timed."""
    call()
    best = 1e30
    for _ in range(n):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best * 1e6


def _muca_us(ctx, L, W, lnW, nsweeps, record):
    spins, E = ctx.muca_start(L, W, 3, start=1)
    ws = ctx.muca_workspace(L, W)
    H = torch.zeros(L * L // 2 + 1, dtype=torch.int64, device="cuda")
    return _us(lambda: ctx.muca_sweeps(L, spins, E, lnW, 3, 0, nsweeps, record, H, ws)) / nsweeps


def _slope(L, b):
    return -b * (4.0 * np.arange(L * L // 2 + 1) - 2.0 * L * L)


# us per sweep without counting, one lane per walker and four: L = 4 15 and 61,
# L = 8 21 and 43, L = 24 238 and 335
@pytest.mark.parametrize("L,W,bound", [(4, 1 << 20, 30.0), (8, 1 << 18, 32.0), (24, 1 << 18, 290.0)])
def test_many_walkers_without_counting(ctx, L, W, bound):
    assert _muca_us(ctx, L, W, _slope(L, 0.3), 20 if L < 24 else 6, False) < bound


# a table with a threshold of 2^32 - 1 takes 1.2 times an ordinary one's time, a
# kernel with one lane per walker 2.8 to 4.3 times
@pytest.mark.parametrize("L", [32, 64, 128])
def test_threshold_next_to_one(ctx, L):
    W, n = 4096, 4 if L < 128 else 1
    plain = _muca_us(ctx, L, W, _slope(L, 0.4), n, True)
    assert _muca_us(ctx, L, W, -3e-10 * np.arange(L * L // 2 + 1), n, True) < 1.8 * plain


# us per sweep of 256 lattices, whole 13.5 and 12.0, half by half 49 and 61
@pytest.mark.parametrize("shape,J", [((32, 32, 160), False), ((32, 5440), True)])
def test_many_wide_lattices(ctx, shape, J):
    n, count = 20, 256
    g = mcs.make_geom(len(shape), shape, count=count)
    lat = mcs.lattice_tensor(g)
    ctx.init(g, lat, mcs.HOT, 3)
    Jd = None
    if J:
        Jd = torch.empty(g.dims * g.N, dtype=torch.int8, device="cuda")
        ctx.couplings(g, Jd, 5)
    EM = torch.empty((n, count, 2), dtype=torch.int64, device="cuda")
    assert _us(lambda: ctx.sweep(g, lat, 0.3, 3, n, J=Jd, EM=EM)) / n < 25.0
