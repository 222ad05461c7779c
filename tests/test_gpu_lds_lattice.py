"""Whole lattices swept in a workgroup's LDS (population annealing and parallel
tempering), bit for bit against the oracle where the layout can go wrong: the
word shapes (four copies of an 8-site colour, several rows to a word, one to
eight words per row, a row of three), the tie queue past its capacity, one, two
and four waves per workgroup, and ragged last workgroups."""
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


# workgroups: 2 replicas of L = 512 (16 words per lane, more ties than the queue
# holds), 2100 and 4200 of L = 64 (two waves, one wave per workgroup), ...
@pytest.mark.parametrize("Ls,R,theta,dbeta,nsteps", [([512], 2, 1, 0.0003, 2), ([192, 320], 3, 2, 0.001, 2),
                                                     ([256, 4, 8], 33, 2, 0.001, 2), ([64], 8400, 1, 0.02, 1),
                                                     ([64], 16801, 1, 0.02, 1), ([4], 300001 // 7, 3, 0.3, 3),
                                                     ([8, 16, 32], 777, 3, 0.05, 3)])
def test_annealing(ctx, Ls, R, theta, dbeta, nsteps):
    beta = np.arange(nsteps + 1) * dbeta
    pops = ctx.pa_population_tensors(Ls, R)
    res = ctx.pa_anneal(Ls, R, theta, 17, beta, pops)
    torch.cuda.synchronize()
    for p, L in enumerate(Ls):
        op = oracle.PAPopulation(L, R, p, 17).advance(beta, theta, nsteps)
        assert np.array_equal(res["lnZ"][p], np.array(op.lnZ[-(nsteps + 1):])), L
        for s in range(nsteps + 1):
            assert np.array_equal(res["hist"][p][s], op.hist[len(op.hist) - nsteps - 1 + s]), (L, s)
        assert np.array_equal(pops[p][:R * L * L].cpu().numpy(), op.spins), L


@pytest.mark.parametrize("L,nT,n_sets,theta", [(4, 7, 3, 3), (8, 5, 13, 2), (192, 3, 1, 2), (256, 2, 2, 1),
                                               (16, 3, 1400, 1), (64, 3, 5, 3)])
def test_tempering(ctx, L, nT, n_sets, theta):
    beta = [0.40 + 0.6 * i / L for i in range(nT)]
    rounds = 3
    st = ctx.pt_state(L, nT, n_sets, 41)
    E_at = ctx.pt_run(L, beta, theta, 41, st, 0, rounds)
    torch.cuda.synchronize()
    spins = st["spins"].cpu().numpy()
    for s in range(0, n_sets, max(1, n_sets // 20)):
        ref = oracle.pt_run(2, L, beta, 41, rounds, theta, pt_set=s)
        assert np.array_equal(E_at[:, s, :], ref["E_at"]), s
        assert list(st["temp_of"][s]) == ref["temp_of"], s
        for r in range(nT):
            assert np.array_equal(spins[s * nT + r], ref["spins"][r]), (s, r)
