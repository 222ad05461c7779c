"""Tuned geometries: a call is not slower for it, its results are the oracle's,
and a geometry whose calls choose their own shape is left out of a saved file
and takes a shape that is set afterwards."""
import time

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
mcs = pytest.importorskip("paper_1709_04394_amd")


@pytest.fixture
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return mcs.Context(0)


def _call(ctx, shape, n, rule, count):
    g = mcs.make_geom(len(shape), shape, count=count)
    lat = mcs.lattice_tensor(g)
    ctx.init(g, lat, mcs.HOT, 9)
    ws = torch.empty(ctx.sweep_workspace_bytes(g), dtype=torch.uint8, device="cuda")
    EM = torch.empty((n, count, 2), dtype=torch.int64, device="cuda")

    def run():
        ctx.sweep(g, lat, 0.3, 9, n, rule=rule, EM=EM, ws=ws)

    run()
    torch.cuda.synchronize()
    first = lat.cpu().numpy(), EM.cpu().numpy()
    best = 1e30
    for _ in range(9):
        torch.cuda.synchronize()
        t = time.perf_counter()
        run()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return first, best


# whole in a workgroup 1.1 us per sweep of 64^2 and 1.5 of 64 x 16 x 16, tiles at
# least 2.5 and 4.5
@pytest.mark.parametrize("shape,rule", [((64, 64), 0), ((64, 16, 16), 1)])
def test_tuned_is_not_slower(ctx, tmp_path, shape, rule):
    n = 100
    untuned, t0 = _call(ctx, shape, n, rule, 1)
    g = mcs.make_geom(len(shape), shape)
    plan = ctx.tune_sweep(g, mcs.lattice_tensor(g), mcs.lattice_tensor(g), 0.3, sweeps=8, rule=rule)
    assert plan == ctx.get_tile_plan(g)
    tuned, t1 = _call(ctx, shape, n, rule, 1)
    assert np.array_equal(untuned[0], tuned[0]) and np.array_equal(untuned[1], tuned[1])
    s = oracle.init(len(shape), shape, oracle.HOT, 9, 0)
    em = oracle.sweep(len(shape), shape, s, 0.3, 9, 0, 0, n, rule=rule)
    assert np.array_equal(tuned[0][0], s) and np.array_equal(tuned[1][:, 0], em)
    assert t1 < 1.4 * t0
    path = str(tmp_path / "shapes.txt")
    ctx.save_launch_shapes(path)
    assert not [x for x in open(path).read().splitlines() if x.startswith("tile ")]
    # a shape that is set holds, and is saved
    ctx.set_tile_plan(g, 4, 2, 256)
    assert ctx.get_tile_plan(g) == (4, 2, 256)
    fixed, _ = _call(ctx, shape, n, rule, 1)
    assert np.array_equal(fixed[0], tuned[0]) and np.array_equal(fixed[1], tuned[1])
    ctx.save_launch_shapes(path)
    assert [x for x in open(path).read().splitlines() if x.startswith("tile ")]


@pytest.mark.parametrize("shape,rule,count", [((64, 6), 0, 2), ((1024, 512), 0, 2), ((128, 32, 36), 1, 2), ((64, 4, 4), 0, 3)])
def test_tuned_results(ctx, shape, rule, count):
    g = mcs.make_geom(len(shape), shape, count=count)
    ctx.tune_sweep(g, mcs.lattice_tensor(g), mcs.lattice_tensor(g), 0.3, sweeps=4, rule=rule)
    (lat, EM), _ = _call(ctx, shape, 5, rule, count)
    for l in range(count):
        s = oracle.init(len(shape), shape, oracle.HOT, 9, l)
        em = oracle.sweep(len(shape), shape, s, 0.3, 9, l, 0, 5, rule=rule)
        assert np.array_equal(lat[l], s) and np.array_equal(EM[:, l], em), l
