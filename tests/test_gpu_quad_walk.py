"""The sequential walker kernels with four lanes per walker (multicanonical
and Wang-Landau), bit for bit against the oracle where their layout can go
wrong: walkers that do not fill a wave or a workgroup, several waves sharing a
table, every row shape (one short word, 24-bit words, one to four whole words,
the one-word wrap-around), the 16-bit counts at L = 128 past their flushes,
a threshold of 2^32 - 1 (the other kernel), and estimates far apart."""
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


def _muca(ctx, L, W, lnW, nsw, record, seed, sweep0=0, start=1):
    spins, E = ctx.muca_start(L, W, seed, start=start)
    H = torch.full((L * L // 2 + 1,), 7, dtype=torch.int64, device="cuda")
    ctx.muca_sweeps(L, spins, E, lnW, seed, sweep0, nsw, record, H=H)
    torch.cuda.synchronize()
    os_, oE = oracle.muca_start(L, W, seed, start)
    oH = oracle.muca_sweeps(L, os_, oE, lnW, seed, sweep0, nsw, record)
    assert np.array_equal(E.cpu().numpy(), oE)
    assert np.array_equal(H.cpu().numpy() - 7, oH if record else 0 * oH)
    assert np.array_equal(spins.cpu().numpy().reshape(-1), os_)


def _slope(L, b):
    return -b * (4.0 * np.arange(L * L // 2 + 1) - 2.0 * L * L)


@pytest.mark.parametrize("L", [4, 8, 12, 16, 24, 32, 48, 64, 96, 128])
@pytest.mark.parametrize("W", [1, 15, 33])
def test_muca_partial_waves(ctx, L, W):
    # sweep numbers crossing 2^32
    _muca(ctx, L, W, _slope(L, 0.3), 2, W != 15, 3 + L + W, sweep0=(1 << 32) - 1)


@pytest.mark.parametrize("L,W", [(8, 4113), (8, 16400), (12, 9000), (16, 8193), (128, 4097)])
def test_muca_shared_tables(ctx, L, W):
    # 2 or 4 waves per workgroup, the last workgroup with empty waves
    _muca(ctx, L, W, _slope(L, 0.42), 1, True, 11 + L, start=0)


@pytest.mark.parametrize("L,W", [(4, 40), (16, 40), (64, 20)])
@pytest.mark.parametrize("step", [3e-10, 6e-10])
def test_muca_threshold_next_to_one(ctx, L, W, step):
    # ln W falling by 3e-10 per level: thresholds 2^32 - 1 and 2^32 - 2
    _muca(ctx, L, W, -step * np.arange(L * L // 2 + 1), 2, True, 29)


def test_muca_steep_weights(ctx):
    # thresholds of 1 (accepted by r32 = 0 alone) in both directions
    lnW = np.cumsum(np.random.default_rng(2).normal(0.0, 30.0, 16 * 16 // 2 + 1))
    _muca(ctx, 16, 100, lnW, 3, True, 5)


def _wl(ctx, L, lo, hi, M, G0, inc, nsw, seed=31, sweep0=(1 << 32) - 2):
    wmax = G0.shape[1]
    W = len(lo) * M
    s, E = ctx.win_drive(L, lo, hi, M, seed)
    so, Eo = s.cpu().numpy(), E.cpu().numpy()
    G = torch.from_numpy(G0.copy()).cuda()
    H = torch.zeros((W, wmax), dtype=torch.int32, device="cuda")
    fl = torch.full((W,), -1, dtype=torch.int32, device="cuda")
    ctx.wl_sweeps(L, lo, hi, M, inc, [1] * len(lo), seed, sweep0, nsw, s, E, G, H, fl)
    torch.cuda.synchronize()
    Go, Ho = G0.copy(), np.zeros((W, wmax), dtype=np.uint32)
    oracle.wl_sweeps(L, lo, hi, M, inc, [1] * len(lo), seed, sweep0, nsw, so, Eo, Go, Ho)
    assert np.array_equal(s.cpu().numpy(), so)
    assert np.array_equal(E.cpu().numpy(), Eo)
    assert np.array_equal(G.cpu().numpy(), Go)
    assert np.array_equal(H.cpu().numpy().view(np.uint32), Ho)
    got = fl.cpu().numpy()
    for w in range(W):
        assert got[w] == int(oracle.wl_flat(Ho[w], lo[w // M], hi[w // M], 0.8)), w


WL_SHAPES = [(4, [0], [8]), (8, [0, 6], [7, 32]), (12, [0, 30], [40, 72]), (16, [0, 60], [61, 128]),
             (24, [0, 150], [160, 288]), (48, [0, 180, 350, 520, 690, 860, 1030],
                                          [190, 360, 530, 700, 870, 1040, 1152])]


@pytest.mark.parametrize("L,lo,hi", WL_SHAPES)
def test_wl_row_shapes(ctx, L, lo, hi):
    wmax = max(h - l for l, h in zip(lo, hi)) + 1
    G0 = np.random.default_rng(L).integers(0, 2 << 32, size=(64 * len(lo), wmax)).astype(np.int64)
    _wl(ctx, L, lo, hi, 64, G0, [1 << (32 - 3 * (i % 8)) for i in range(len(lo))], 3)


@pytest.mark.parametrize("gmax", [1, 1 << 17, 1 << 40, 1 << 60])
@pytest.mark.parametrize("inc", [0, 1, 1 << 32])
def test_wl_estimate_ranges(ctx, gmax, inc):
    # equal estimates, differences around the margin of the FP32 test, and far
    # beyond any acceptance, of either sign
    L, lo, hi = 32, [0, 160, 330], [180, 340, 512]
    G0 = np.random.default_rng(7).integers(-gmax, gmax, size=(3 * 64, 183)).astype(np.int64)
    _wl(ctx, L, lo, hi, 64, G0, [inc] * 3, 2)
