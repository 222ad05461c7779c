"""Double-checkerboard launches whose tied words one wave settles for the whole
workgroup (tiles of 128, 1024 workgroups or more), and those just beside the
rule: sampled lattices and every sweep's (E, M) against the oracle."""
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


@pytest.mark.parametrize("L,T,count,hits", [(256, 128, 512, 3), (256, 128, 511, 2), (768, 128, 57, 2),
                                            (128, 64, 600, 3), (512, 256, 512, 1)])
def test_pooled_ties(ctx, L, T, count, hits):
    seed, r0, beta, nsw = 61, 3, 0.43, 2
    g = mcs.make_geom(2, L, count=count)
    lat = mcs.lattice_tensor(g)
    ctx.init(g, lat, mcs.HOT, seed, r0)
    EM = torch.empty((nsw, count, 2), dtype=torch.int64, device="cuda")
    ws = torch.empty(ctx.dcb_workspace_bytes(g), dtype=torch.uint8, device="cuda")
    ctx.sweep_dcb(g, lat, beta, seed, nsw, T, hits, sweep0=5, replica0=r0, EM=EM, ws=ws)
    torch.cuda.synchronize()
    for l in (0, count // 2, count - 1):
        s = oracle.init(2, L, oracle.HOT, seed, r0 + l)
        ref = oracle.sweep_dcb(L, s, beta, seed, r0 + l, 5, nsw, T, hits)
        assert np.array_equal(lat[l].cpu().numpy(), np.asarray(s).reshape(-1)), l
        assert np.array_equal(EM[:, l, :].cpu().numpy(), ref), l
