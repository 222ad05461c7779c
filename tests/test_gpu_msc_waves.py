"""Multi-spin-coded half-sweeps where a wave walks many tasks: more than the
bit-sliced counters are summed over at once (2D) and several tie queues' worth
of ties (3D heat-bath), sampled replicas against the int8 oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
mcs = pytest.importorskip("paper_1709_04394_amd")


@pytest.mark.parametrize("dims,shape,rule,beta,lanes", [(2, (4096, 4228), 0, 0.44, (0, 3, 4, 63)),
                                                        (2, (4096, 4228), 1, 0.44, (7, 40)),
                                                        (3, (128, 370, 366), 1, 0.2216546, (2, 33)),
                                                        (3, (128, 370, 366), 0, 0.2216546, (5, 62))])
def test_many_tasks_per_wave(dims, shape, rule, beta, lanes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = mcs.Context(0)
    g = mcs.make_geom(dims, shape, layout=mcs.MSC64)
    w = mcs.lattice_tensor(g)
    ctx.init(g, w, mcs.HOT, 7, 0)
    EM = torch.empty((1, 64, 2), dtype=torch.int64, device="cuda")
    ctx.sweep(g, w, beta, 7, 1, sweep0=(1 << 32) + 5, rule=rule, EM=EM)
    torch.cuda.synchronize()
    words, em = w.cpu().numpy().view(np.uint64).reshape(-1), EM.cpu().numpy()
    for b in lanes:
        s = oracle.init(dims, shape, oracle.HOT, 7, b)
        ref = oracle.sweep(dims, shape, s, beta, 7, b, (1 << 32) + 5, 1, rule=rule)
        assert np.array_equal(em[:, b, :], ref), b
        assert np.array_equal(np.where((words >> np.uint64(b)) & np.uint64(1), -1, 1).astype(np.int8), s), b


@pytest.mark.parametrize("dims,shape,count", [(2, (128, 64), 2), (2, (512, 384), 2), (2, (1024, 512), 1),
                                              (3, (128, 16, 24), 3), (3, (256, 36, 34), 1)])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("measure", [True, False])
def test_waves_per_workgroup(dims, shape, count, rule, measure):
    """Workgroups of 4, 8 and 16 waves that measure, and of 4 that do not."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = mcs.Context(0)
    beta, nsw = (0.44, 0.2216546)[dims - 2], 3
    g = mcs.make_geom(dims, shape, layout=mcs.MSC64, count=count)
    w = mcs.lattice_tensor(g)
    ctx.init(g, w, mcs.HOT, 8, 0)
    EM = torch.empty((nsw, 64 * count, 2), dtype=torch.int64, device="cuda") if measure else None
    ctx.sweep(g, w, beta, 8, nsw, rule=rule, EM=EM)
    torch.cuda.synchronize()
    words = w.cpu().numpy().view(np.uint64).reshape(count, -1)
    for l in range(count):
        for b in (1, 30, 63):
            s = oracle.init(dims, shape, oracle.HOT, 8, 64 * l + b)
            ref = oracle.sweep(dims, shape, s, beta, 8, 64 * l + b, 0, nsw, rule=rule)
            if measure:
                assert np.array_equal(EM[:, 64 * l + b, :].cpu().numpy(), ref), (l, b)
            assert np.array_equal(np.where((words[l] >> np.uint64(b)) & np.uint64(1), -1, 1).astype(np.int8), s), (l, b)
