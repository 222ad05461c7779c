"""Half-sweeps in global memory of int8 lattices with rows of 32 sites or more,
where their chunks can go wrong: rows of 16 sites a colour, of one more, of one
fewer than two chunks (random bits from two blocks, shifted; a last chunk that
overlaps the one before), rows that hold whole chunks, unaligned rows, several
lattices, more chunks than threads, each rule, with and without couplings, with
and without (E, M).  Spins and per-sweep (E, M) against the oracle, bit for
bit; a canary after the lattices stays as it was."""
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


def _check(ctx, dims, shape, count, rule, J, measure, nsw=3, sweep0=(1 << 32) - 1):
    seed, r0, beta = 37, 6, 0.45 if dims == 2 else 0.25
    g = mcs.make_geom(dims, shape, count=count)
    n = count * g.N
    buf = torch.full((n + 4096,), 77, dtype=torch.int8, device="cuda")
    lat = buf[:n].view(count, g.N)
    ctx.init(g, lat, mcs.HOT, seed, r0)
    Jt = None
    if J:
        Jt = torch.empty(dims * g.N, dtype=torch.int8, device="cuda")
        ctx.couplings(g, Jt, seed + 1)
    EM = torch.full((nsw, count, 2), -5, dtype=torch.int64, device="cuda") if measure else None
    ctx.sweep(g, lat, beta, seed, nsw, sweep0=sweep0, replica0=r0, rule=rule, J=Jt, EM=EM, ws=None)
    torch.cuda.synchronize()
    assert bool((buf[n:] == 77).all())
    Jh = oracle.couplings(dims, shape, seed + 1) if J else None
    for l in range(count):
        s = oracle.init(dims, shape, oracle.HOT, seed, r0 + l)
        ref = oracle.sweep(dims, shape, s, beta, seed, r0 + l, sweep0, nsw,
                           rule=oracle.HEATBATH if rule else oracle.METROPOLIS, J=Jh)
        assert np.array_equal(lat[l].cpu().numpy(), np.asarray(s).reshape(-1)), ("spins", l)
        if measure:
            assert np.array_equal(EM[:, l, :].cpu().numpy(), ref), ("EM", l)


@pytest.mark.parametrize("dims,shape,count,J", [
    (2, (32, 16390), 1, False),     # one chunk per row
    (2, (34, 3100), 2, False),      # 17 sites a colour
    (2, (46, 2300), 1, False),
    (2, (62, 1700), 1, False),      # 31
    (2, (64, 1700), 1, False),      # 32: blocks and chunks agree
    (2, (1000, 110), 3, False),
    (2, (50, 900), 2, True),
    (2, (96, 500), 1, True),
    (3, (34, 40, 80), 1, False),
    (3, (34, 34, 34), 2, True),
    (3, (64, 10, 60), 1, True),
])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("measure", [True, False])
def test_chunks_of_rows(ctx, dims, shape, count, J, rule, measure):
    _check(ctx, dims, shape, count, rule, J, measure)


@pytest.mark.parametrize("rule,J", [(1, False), (0, True)])
def test_more_chunks_than_threads(ctx, rule, J):
    # 1.2 million chunks: several per thread
    _check(ctx, 2, (4100, 9000), 1, rule, J, True, nsw=1)


def test_lattices_of_different_temperatures(ctx):
    # mc_sweep_betas without tiles: each lattice alone, (E, M) rows interleaved
    shape, count, seed, nsw = (330, 350), 3, 5, 2
    betas = [0.3, 0.44, 0.6]
    g = mcs.make_geom(2, shape, count=count)
    lat = mcs.lattice_tensor(g)
    ctx.init(g, lat, mcs.HOT, seed, 0)
    EM = torch.full((nsw, count, 2), -5, dtype=torch.int64, device="cuda")
    ctx.sweep_betas(g, lat, betas, seed, nsw, rule=mcs.HEATBATH, EM=EM)
    torch.cuda.synchronize()
    for l in range(count):
        s = oracle.init(2, shape, oracle.HOT, seed, l)
        ref = oracle.sweep(2, shape, s, betas[l], seed, l, 0, nsw, rule=oracle.HEATBATH)
        assert np.array_equal(lat[l].cpu().numpy(), np.asarray(s).reshape(-1)), l
        assert np.array_equal(EM[:, l, :].cpu().numpy(), ref), l
