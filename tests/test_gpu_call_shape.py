"""2D calls without a set or tuned tile plan pick their launch shape by extents,
count and number of sweeps: bit for bit against the oracle at the edges of the
choice (few rows, rows wider than a workgroup, band heights that do not divide
the lattice, one sweep, more sweeps than a launch takes, many lattices), with
and without (E, M)."""
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


@pytest.mark.parametrize("shape,count,nsweeps", [((64, 4), 1, 1), ((64, 4), 3, 19), ((64, 6), 1, 2), ((64, 64), 1, 10),
                                                 ((128, 74), 2, 7), ((192, 100), 70, 3), ((64, 64), 300, 9),
                                                 ((64, 18), 600, 5), ((4160, 20), 1, 5), ((12352, 10), 2, 3),
                                                 ((16384, 6), 1, 4), ((576, 1030), 1, 8), ((1024, 1024), 1, 17)])
def test_call_matches_oracle(ctx, shape, count, nsweeps):
    beta, seed, sweep0, rep0 = 0.43, 13, (1 << 32) - 3, 5
    g = mcs.make_geom(2, shape, count=count)
    ws = torch.empty(ctx.sweep_workspace_bytes(g), dtype=torch.uint8, device="cuda")
    out = []
    for measure in (True, False):
        spins = mcs.lattice_tensor(g)
        ctx.init(g, spins, mcs.HOT, seed, rep0)
        EM = torch.empty((nsweeps, count, 2), dtype=torch.int64, device="cuda") if measure else None
        ctx.sweep(g, spins, beta, seed, nsweeps, sweep0=sweep0, replica0=rep0, EM=EM, ws=ws)
        torch.cuda.synchronize()
        out.append(spins.cpu().numpy())
        if measure:
            em = EM.cpu().numpy()
    assert np.array_equal(out[0], out[1])
    for l in range(0, count, max(1, count // 8)):
        s = oracle.init(2, shape, oracle.HOT, seed, rep0 + l)
        ref = oracle.sweep(2, shape, s, beta, seed, rep0 + l, sweep0, nsweeps)
        assert np.array_equal(em[:, l, :], ref), l
        assert np.array_equal(out[0][l], s), l


@pytest.mark.parametrize("shape,count,nsweeps", [((64, 4, 4), 1, 3), ((64, 4, 6), 5, 9), ((64, 10, 34), 1, 1),
                                                 ((128, 22, 46), 2, 5), ((64, 64, 64), 1, 13), ((192, 36, 8), 40, 4),
                                                 ((1024, 4, 12), 1, 6), ((4096, 4, 4), 1, 2)])
@pytest.mark.parametrize("rule,J", [(0, False), (1, True)])
def test_call_3d_matches_oracle(ctx, shape, count, nsweeps, rule, J):
    beta, seed, sweep0, rep0 = 0.3, 17, (1 << 32) - 2, 3
    g = mcs.make_geom(3, shape, count=count)
    ws = torch.empty(ctx.sweep_workspace_bytes(g), dtype=torch.uint8, device="cuda")
    Jd = Jh = None
    if J:
        Jd = torch.empty(3 * g.N, dtype=torch.int8, device="cuda")
        ctx.couplings(g, Jd, 23)
        Jh = Jd.cpu().numpy()
    spins = mcs.lattice_tensor(g)
    ctx.init(g, spins, mcs.HOT, seed, rep0)
    EM = torch.empty((nsweeps, count, 2), dtype=torch.int64, device="cuda")
    ctx.sweep(g, spins, beta, seed, nsweeps, sweep0=sweep0, replica0=rep0, rule=rule, J=Jd, EM=EM, ws=ws)
    torch.cuda.synchronize()
    got, em = spins.cpu().numpy(), EM.cpu().numpy()
    for l in range(0, count, max(1, count // 4)):
        s = oracle.init(3, shape, oracle.HOT, seed, rep0 + l)
        ref = oracle.sweep(3, shape, s, beta, seed, rep0 + l, sweep0, nsweeps, rule=rule, J=Jh)
        assert np.array_equal(em[:, l, :], ref), l
        assert np.array_equal(got[l], s), l
