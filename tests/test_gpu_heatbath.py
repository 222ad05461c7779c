"""Heat-bath threshold planes from mirrored classes and from all classes: fields
where every product p 2^32 is an ordinary number, where the two outer ones are 1
and 2^32 or 0 and 2^32, beta = 0 (all 2^31), beta = 1e-12 (2^31 + 1 and 2^31),
and p = 200/256 at h = 2, whose threshold's top byte is on the edge.  Every path
that draws planes, spins and per-sweep (E, M) against the oracle, bit for bit."""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
mcs = pytest.importorskip("paper_1709_04394_amd")

EDGE = math.log(200 / 56) / 4  # 1 / (1 + exp(-2 beta 2)) = 200/256


@pytest.mark.parametrize("beta", [0.0, 1e-12, 0.22, EDGE, 2.0, 100.0])
@pytest.mark.parametrize("dims,shape,msc,ws,J", [
    (3, (64, 24, 26), False, True, True),    # fused tiles
    (3, (64, 24, 26), False, True, False),
    (2, (1030, 140), False, False, False),   # half-sweeps in global memory
    (3, (64, 50, 44), False, False, True),
    (2, (50, 46), False, False, False),      # one workgroup
    (3, (64, 12, 10), False, True, False),
    (3, (16, 10, 12), False, False, True),
    (2, (128, 20), True, False, False),      # 64 replicas to a word
    (3, (128, 6, 8), True, False, True),
])
def test_threshold_planes(dims, shape, msc, ws, J, beta):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = mcs.Context(0)
    nsw, seed, sweep0 = 4, 21, (1 << 32) - 2
    g = mcs.make_geom(dims, shape, layout=mcs.MSC64 if msc else mcs.INT8)
    lat = mcs.lattice_tensor(g)
    ctx.init(g, lat, mcs.HOT, seed, 0)
    Jt = None
    if J:
        Jt = torch.empty(dims * g.N, dtype=torch.int8, device="cuda")
        ctx.couplings(g, Jt, seed + 1)
    Jh = oracle.couplings(dims, shape, seed + 1) if J else None
    EM = torch.empty((nsw, 64 if msc else 1, 2), dtype=torch.int64, device="cuda")
    w = torch.empty(ctx.sweep_workspace_bytes(g), dtype=torch.uint8, device="cuda") if ws else None
    ctx.sweep(g, lat, beta, seed, nsw, sweep0=sweep0, rule=1, J=Jt, EM=EM, ws=w)
    torch.cuda.synchronize()
    got = lat.cpu().numpy().reshape(-1)
    for r in (0, 5, 62) if msc else (0,):
        s = oracle.init(dims, shape, oracle.HOT, seed, r)
        ref = oracle.sweep(dims, shape, s, beta, seed, r, sweep0, nsw, rule=oracle.HEATBATH, J=Jh)
        mine = np.where((got.view(np.uint64) >> np.uint64(r)) & np.uint64(1), -1, 1).astype(np.int8) if msc else got
        assert np.array_equal(mine, np.asarray(s).reshape(-1)), r
        assert np.array_equal(EM[:, r, :].cpu().numpy(), ref), r
