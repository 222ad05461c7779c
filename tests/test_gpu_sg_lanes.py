"""The realisation-coded half-sweep where its work division can go wrong:
rows shorter than a wave's 64 sites that do not divide them (several rows and
planes in one task), rows longer than a task, lattices of one task and of more
tasks than the launch has waves (several sums of the counters per wave), and
numbers of workgroups that are not multiples of eight.  Spins and per-sweep
(E, M) of sampled realisations against the oracle, bit for bit."""
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


@pytest.mark.parametrize("dims,shape,count,nsw,lanes", [
    (2, (4, 32), 3, 4, (0, 1, 63)),            # one task: 32 rows of two sites a colour
    (3, (4, 4, 8), 2, 4, (5, 62)),             # a task over several planes
    (3, (6, 8, 16), 5, 3, (0, 33)),            # three sites a colour: 64 / 3 rows
    (3, (48, 4, 4), 1, 3, (0, 31, 32)),        # rows of 24
    (2, (96, 8), 2, 3, (0, 40)),               # rows of 48
    (2, (130, 64), 1, 3, (2, 63)),             # rows of 65
    (2, (1024, 768), 2, 2, (7,)),              # more tasks than waves
    (2, (16, 96000), 1, 2, (17,)),             # the same, eight rows to a task
])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("measure", [True, False])
def test_work_division(ctx, dims, shape, count, nsw, lanes, rule, measure):
    seed, r0, z0, beta = 29, 4, 2, 0.7
    g = mcs.make_geom(dims, shape, layout=mcs.MSC64, count=count)
    w = mcs.lattice_tensor(g)
    ctx.init(g, w, mcs.HOT, seed, r0)
    J = torch.empty((count, dims * g.N), dtype=torch.int64, device="cuda")
    ctx.couplings_msc64(g, J, seed + 1, z0)
    EM = torch.empty((nsw, count * 64, 2), dtype=torch.int64, device="cuda") if measure else None
    ctx.sweep_sg_msc64(g, w, J, beta, seed, nsw, sweep0=3, replica0=r0, rule=rule, EM=EM)
    torch.cuda.synchronize()
    wh = w.cpu().numpy().view(np.uint64).reshape(count, -1)
    orule = oracle.HEATBATH if rule else oracle.METROPOLIS
    for l in {0, count - 1}:
        for b in lanes:
            s = oracle.init(dims, shape, oracle.HOT, seed, r0 + 64 * l + b)
            Jr = oracle.couplings(dims, shape, seed + 1, z0 + 64 * l + b)
            ref = oracle.sweep(dims, shape, s, beta, seed, r0 + l, 3, nsw, rule=orule, J=Jr)
            got = np.where((wh[l] >> np.uint64(b)) & np.uint64(1), -1, 1).astype(np.int8)
            assert np.array_equal(got, s.reshape(-1)), ("spins", l, b)
            if measure:
                assert np.array_equal(EM[:, 64 * l + b, :].cpu().numpy(), ref), ("EM", l, b)
