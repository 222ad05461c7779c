"""Tempering runs in several calls of equal length (which launch the graph of
the first with their own first round) and exchange thresholds beyond the
stored rows: pairs of temperatures so far apart that the threshold of a likely
energy difference is 1, or 0, and so close that a row holds every difference.
Against the oracle, bit for bit."""
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


@pytest.mark.parametrize("L,beta,theta,calls,rounds", [
    (16, [0.30, 0.35, 0.40, 0.45], 2, 3, 5),
    (16, [0.05, 0.40, 0.60, 3.0, 40.0], 1, 3, 4),      # thresholds 1 and 0
    (8, [0.1, 1.0, 20.0], 1, 2, 9),
    (32, [0.42, 0.42 + 1e-9, 0.42 + 2e-4], 1, 2, 4),   # whole rows
    (64, [0.40, 0.41, 0.43, 0.50], 1, 2, 3),
])
def test_equal_calls_and_far_temperatures(ctx, L, beta, theta, calls, rounds):
    seed, n_sets = 53, 2
    st = ctx.pt_state(L, len(beta), n_sets, seed)
    ws = torch.empty(ctx.pt_workspace_bytes(L, beta, n_sets, theta, rounds), dtype=torch.uint8, device="cuda")
    E = []
    for k in range(calls):
        E.append(ctx.pt_run(L, beta, theta, seed, st, k * rounds, rounds, ws=ws))
        ws.fill_(0x3C)
        torch.cuda.synchronize()
    E = np.concatenate(E, axis=0)
    spins = st["spins"].cpu().numpy()
    for s in range(n_sets):
        ref = oracle.pt_run(2, L, beta, seed, calls * rounds, theta, pt_set=s)
        assert np.array_equal(E[:, s, :], ref["E_at"]), s
        assert list(st["temp_of"][s]) == ref["temp_of"], s
        assert list(st["accepted"][s]) == ref["accepted"], s
        for r in range(len(beta)):
            assert np.array_equal(spins[s * len(beta) + r], ref["spins"][r]), (s, r)


def test_rows_cut_where_the_threshold_is_constant():
    """The stored rows end, and the threshold turns to 0, where libm says so."""
    for d in (0.2 / 31, 0.01, 0.35, 2.4, 37.0):
        m = np.arange(1, 4097, dtype=np.float64)
        T = np.array([int(np.ceil(np.ldexp(np.exp(-d * 4 * k), 32))) for k in m])
        x = -d * 4 * m
        assert np.all(T[(x < -22.5) & (x > -744.0)] == 1)
        assert np.all(T[x < -746.0] == 0)
