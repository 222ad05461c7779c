"""Sweeps of small int8 lattices held whole as bits in a workgroup, where the
words of their sites can go wrong: fewer sites of a colour than a word, numbers
that are not multiples of 32 (a last word with fewer sites, windows round the
end), rows shorter and longer than a word, rows and planes that end inside a
word, one and two words per thread, each rule, with and without couplings, with
and without (E, M), several lattices; and lattices of the fused tiles' shapes
that take this route.  Spins and per-sweep (E, M) against the oracle, bit for
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


def _check(ctx, dims, shape, count, rule, J, measure, nsw=5, sweep0=(1 << 32) - 2, with_ws=False, beta=None):
    seed, r0 = 41, 9
    beta = (0.45 if dims == 2 else 0.25) if beta is None else beta
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
    ws = torch.empty(max(ctx.sweep_workspace_bytes(g), 1), dtype=torch.uint8, device="cuda") if with_ws else None
    ctx.sweep(g, lat, beta, seed, nsw, sweep0=sweep0, replica0=r0, rule=rule, J=Jt, EM=EM, ws=ws)
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


@pytest.mark.parametrize("dims,shape,count", [
    (2, (4, 4), 3),          # 8 sites of a colour
    (2, (4, 6), 2),          # 12
    (2, (6, 10), 2),         # 30
    (2, (4, 16), 2),         # 32: one whole word of 16 rows
    (2, (6, 22), 1),         # 66: rows of three
    (2, (10, 10), 2),        # 50
    (2, (34, 18), 1),        # rows of 17
    (2, (66, 14), 3),        # rows of 33
    (2, (130, 126), 1),      # rows of 65, several waves
    (2, (256, 170), 1),      # rows of whole words
    (2, (254, 170), 1),
    (3, (4, 4, 4), 2),       # 32 sites of a colour, planes of 8
    (3, (6, 4, 6), 2),       # planes of 12
    (3, (10, 6, 4), 1),      # planes of 30
    (3, (12, 12, 12), 2),
    (3, (32, 10, 12), 1),    # 32-site rows
    (3, (32, 8, 8), 2),
    (3, (30, 26, 22), 1),
])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("J", [False, True])
def test_words_of_any_extents(ctx, dims, shape, count, rule, J):
    _check(ctx, dims, shape, count, rule, J, True)
    if shape[0] < 20:
        _check(ctx, dims, shape, count, rule, J, False, nsw=2)


@pytest.mark.parametrize("dims,shape,J", [
    (2, (300, 330), False),      # two words per thread, the last word short
    (2, (258, 256), False),      # 1032 words
    (2, (32, 4096), False),      # 2^17 sites
    (2, (32, 2100), True),
    (3, (32, 64, 64), True),     # 2^17 sites with couplings
    (3, (50, 40, 50), False),
])
@pytest.mark.parametrize("rule", [0, 1])
def test_two_words_per_thread(ctx, dims, shape, J, rule):
    _check(ctx, dims, shape, 2, rule, J, True, nsw=3)


@pytest.mark.parametrize("dims,shape,rule,J", [
    (2, (64, 64), 0, False), (2, (192, 20), 0, False), (2, (256, 128), 0, False), (3, (64, 8, 6), 1, True),
    (3, (64, 16, 32), 0, False),
    (2, (256, 130), 0, False), (3, (64, 16, 34), 1, True),   # just above: tiles
])
def test_lattices_of_the_tiles_shapes(ctx, dims, shape, rule, J):
    _check(ctx, dims, shape, 2, rule, J, True, nsw=9, with_ws=True)


@pytest.mark.parametrize("dims,shape,J", [(2, (34, 18), False), (2, (64, 64), False), (2, (66, 62), True),
                                          (3, (12, 12, 12), True), (2, (16, 8), False)])
def test_many_lattices(ctx, dims, shape, J):
    """Enough lattices that a thread takes 32 sites: samples against the same
    lattices in a call of three (16 sites), which other tests compare with the
    oracle."""
    seed, count, nsw = 43, 1100, 3
    g = mcs.make_geom(dims, shape, count=count)
    lat = mcs.lattice_tensor(g)
    ctx.init(g, lat, mcs.HOT, seed, 0)
    Jt = None
    if J:
        Jt = torch.empty(dims * g.N, dtype=torch.int8, device="cuda")
        ctx.couplings(g, Jt, seed + 1)
    g3 = mcs.make_geom(dims, shape, count=3)
    few = lat.view(count, -1)[500:503].clone()
    EM = torch.empty((nsw, count, 2), dtype=torch.int64, device="cuda")
    EM3 = torch.empty((nsw, 3, 2), dtype=torch.int64, device="cuda")
    ctx.sweep(g, lat, 0.5, seed, nsw, J=Jt, EM=EM)
    ctx.sweep(g3, few, 0.5, seed, nsw, replica0=500, J=Jt, EM=EM3)
    torch.cuda.synchronize()
    assert torch.equal(lat.view(count, -1)[500:503], few.view(3, -1))
    assert torch.equal(EM[:, 500:503], EM3)


@pytest.mark.parametrize("beta", [0.0, 0.05, 3.0])
@pytest.mark.parametrize("rule", [0, 1])
def test_extreme_temperatures(ctx, beta, rule):
    # beta = 0: thresholds of 2^32 (Metropolis), every draw a comparison with 1/2 (heat-bath)
    _check(ctx, 2, (22, 18), 2, rule, False, True, beta=beta)
    _check(ctx, 3, (6, 8, 10), 1, rule, True, True, beta=beta)


def test_above_two_words_per_thread(ctx):
    # rows of 32 sites above 2^17 sites: half-sweeps
    _check(ctx, 2, (32, 4100), 1, 0, False, True, nsw=2)
