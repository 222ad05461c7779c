"""Lattices of 32-site rows above 2^17 sites: many of them run whole, each in a
workgroup with more words than two per thread, few half by half.  Bit for bit
against the oracle on both sides of the rule, with the last word of a
workgroup's share ragged, up to the largest such lattice, for every rule and
kind of threshold table (beta = 0 is not mirrored)."""
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


@pytest.mark.parametrize("shape,J", [((32, 4098), False), ((32, 4098), True), ((32, 5460), True), ((32, 16384), False),
                                     ((32, 4, 1026), False), ((32, 130, 34), False), ((32, 64, 256), False)])
@pytest.mark.parametrize("rule,beta", [(0, 0.35), (1, 0.35), (1, 0.0)])
@pytest.mark.parametrize("count,measure", [(8, True), (200, True), (200, False)])
def test_rows_of_32(ctx, shape, J, rule, beta, count, measure):
    d, seed, sweep0, rep0, n = len(shape), 61, (1 << 32) - 1, 7, 2
    g = mcs.make_geom(d, shape, count=count)
    spins = mcs.lattice_tensor(g)
    ctx.init(g, spins, mcs.HOT, seed, rep0)
    Jd = Jh = None
    if J:
        Jd = torch.empty(d * g.N, dtype=torch.int8, device="cuda")
        ctx.couplings(g, Jd, 23)
        Jh = Jd.cpu().numpy()
    EM = torch.empty((n, count, 2), dtype=torch.int64, device="cuda") if measure else None
    ctx.sweep(g, spins, beta, seed, n, sweep0=sweep0, replica0=rep0, rule=rule, J=Jd, EM=EM)
    torch.cuda.synchronize()
    for l in (0, count - 1):
        s = oracle.init(d, shape, oracle.HOT, seed, rep0 + l)
        ref = oracle.sweep(d, shape, s, beta, seed, rep0 + l, sweep0, n, rule=rule, J=Jh)
        assert np.array_equal(spins[l].cpu().numpy(), s), l
        if measure:
            assert np.array_equal(EM[:, l].cpu().numpy(), ref), l
