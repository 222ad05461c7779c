"""Ties of lattices swept in LDS, settled by the lane that owns the word where a
wave has one task a half-sweep and from the wave's queue where it has more: one
wave and four waves per workgroup on either side of the rule that chooses them
(6000 workgroups, 1024 words), words of several rows and of a part of one, and
the last task of a wave part full.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
mcs = pytest.importorskip("paper_1709_04394_amd")


@pytest.mark.parametrize("L,G,R", [(64, 4, 23996), (64, 4, 24001),   # 5999 and 6001 workgroups
                                   (128, 1, 5999), (128, 1, 6000),
                                   (16, 1, 6007), (32, 33, 150),     # 528 tasks
                                   (16, 64, 130), (64, 5, 26), (192, 3, 10)])
def test_annealing(L, G, R):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = mcs.Context(0)
    ctx.set_pa_group(L, G)
    beta, theta, nsteps = np.array([0.0, 0.004]), 2, 1
    pops = ctx.pa_population_tensors([L], R)
    res = ctx.pa_anneal([L], R, theta, 23, beta, pops)
    torch.cuda.synchronize()
    op = oracle.PAPopulation(L, R, 0, 23).advance(beta, theta, nsteps)
    assert np.array_equal(res["lnZ"][0], np.array(op.lnZ))
    assert np.array_equal(res["hist"][0][1], op.hist[1])
    assert np.array_equal(pops[0][:R * L * L].cpu().numpy(), op.spins)


@pytest.mark.parametrize("L,nT,n_sets", [(64, 2, 12002), (64, 2, 11998), (32, 3, 7), (128, 2, 3)])
def test_tempering(L, nT, n_sets):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = mcs.Context(0)
    beta, theta, rounds = [0.42 + 0.6 * i / L for i in range(nT)], 2, 2
    st = ctx.pt_state(L, nT, n_sets, 43)
    E_at = ctx.pt_run(L, beta, theta, 43, st, 0, rounds)
    torch.cuda.synchronize()
    spins = st["spins"].cpu().numpy()
    for s in sorted({0, 1, n_sets // 2, n_sets - 1}):
        ref = oracle.pt_run(2, L, beta, 43, rounds, theta, pt_set=s)
        assert np.array_equal(E_at[:, s, :], ref["E_at"]), s
        for r in range(nT):
            assert np.array_equal(spins[s * nT + r], ref["spins"][r]), (s, r)
