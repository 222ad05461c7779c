"""The timed workloads of the engine: what a user has it do, one entry point per
kind, over the sizes of its benchmark, its tests and its own configurations.

A case names a kind and its sizes; `prepare` sets up what a program holds before
the call (lattices, couplings, weights, workspaces, the context), `run` makes one
call as such a program makes it and returns the states and the measurements.
Every pass continues the simulation: sweep numbers advance, as in a long run.
"""
import math

import numpy as np
import torch

import paper_1709_04394_amd as mcs

BETA_C = math.log(1.0 + math.sqrt(2.0)) / 2.0
BETA_C3 = 0.2216546
DEV = "cuda"


# --------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest call: one small lattice for a few sweeps, the size of the
        # smoke run (latency and launches)
        dict(name="sweep2d_64", kind="sweep", dims=2, Lx=64, Ly=64, Lz=1, count=1, rule=0, J=False, nsweeps=10,
             EM=True),
        # a ragged extent, heat-bath: the path of every lattice that is not a
        # multiple of 64 sites wide
        dict(name="sweep2d_1000x750", kind="sweep", dims=2, Lx=1000, Ly=750, Lz=1, count=1, rule=1, J=False,
             nsweeps=10, EM=True),
        # the headline benchmark: three 4096^2 lattices around beta_c, E and M
        # after every sweep
        dict(name="sweep2d_4096x3", kind="sweep", dims=2, Lx=4096, Ly=4096, Lz=1, count=3, rule=0, J=False,
             nsweeps=50, EM=True),
        # four 256^3 heat-bath lattices, two temperatures
        dict(name="sweep3d_256x4", kind="sweep", dims=3, Lx=256, Ly=256, Lz=256, count=4, rule=1, J=False,
             nsweeps=20, EM=True),
        # one spin-glass realisation of 32^3 (low temperature, long series)
        dict(name="ea3d_32", kind="sweep", dims=3, Lx=32, Ly=32, Lz=32, count=1, rule=0, J=True, nsweeps=100,
             EM=True),
        # 64 replicas of a 4096^2 lattice in the bits of a word
        dict(name="msc2d_4096", kind="msc", dims=2, Lx=4096, Ly=4096, Lz=1, count=1, rule=0, nsweeps=4, EM=True),
        # 4096 disorder realisations of 32^3, coded 64 to a word
        dict(name="sg_32x4096", kind="sg", dims=3, Lx=32, Ly=32, Lz=32, count=64, rule=0, nsweeps=20, EM=True),
        # the double checkerboard with ten hits per tile on the headline's lattices
        dict(name="dcb_4096x3_k10", kind="dcb", L=4096, count=3, tile=128, hits=10, nsweeps=5),
        # the first steps of the annealing benchmark: four populations
        dict(name="pa_4x16384", kind="pa", L0=16, L1=32, L2=64, L3=128, R=16384, theta=10, nsteps=8),
        # the tempering benchmark: 128 sets of 32 temperatures
        dict(name="pt_64x32x128", kind="pt", L=64, n_temps=32, n_sets=128, theta=10, rounds=10),
        # multicanonical iterations at the size of the learned-weights runs
        dict(name="muca_64x4096", kind="muca", L=64, walkers=4096, nsweeps=4, record=True),
        # Wang-Landau in windows: the benchmark's 64 windows of 256 walkers
        dict(name="wl_64x64x256", kind="wl", L=64, nwin=64, walkers=256, nsweeps=2),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of step in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999 * step)))
    return int(max(lo, min(hi, int(v) // step * step)))


def _even(rng, lo, hi):
    return _log(rng, lo, hi, 2)


def draw(rng):
    kind = rng.choice(["fused2d", "ragged", "fused3d", "glass", "msc", "sg", "dcb", "pa", "pt", "muca", "wl"])
    if kind == "fused2d":
        Lx, Ly = _log(rng, 64, 8192, 64), _even(rng, 16, 8192)
        count = max(1, min(rng.choice([1, 2, 3, 5, 8]), 48_000_000 // (Lx * Ly)))
        n = max(1, min(rng.randint(1, 60), 2_400_000_000 // (Lx * Ly * count)))
        return dict(kind="sweep", dims=2, Lx=Lx, Ly=Ly, Lz=1, count=count, rule=0, J=False, nsweeps=n,
                    EM=rng.random() < 0.8)
    if kind == "ragged":
        Lx, Ly = _even(rng, 10, 1400), _even(rng, 10, 1400)
        if Lx % 64 == 0:
            Lx += 2
        n = max(1, min(rng.randint(1, 20), 10_000_000 // (Lx * Ly)))
        return dict(kind="sweep", dims=2, Lx=Lx, Ly=Ly, Lz=1, count=rng.choice([1, 1, 2]), rule=rng.randint(0, 1),
                    J=rng.random() < 0.3, nsweeps=n, EM=rng.random() < 0.7)
    if kind == "fused3d":
        Lx, Ly, Lz = 64 * rng.randint(1, 4), _even(rng, 16, 256), _even(rng, 16, 256)
        count = rng.choice([1, 2, 4])
        n = max(1, min(rng.randint(1, 40), 1_300_000_000 // (Lx * Ly * Lz * count)))
        return dict(kind="sweep", dims=3, Lx=Lx, Ly=Ly, Lz=Lz, count=count, rule=rng.randint(0, 1),
                    J=rng.random() < 0.4, nsweeps=n, EM=rng.random() < 0.8)
    if kind == "glass":
        return dict(kind="sweep", dims=3, Lx=32, Ly=_even(rng, 8, 36), Lz=_even(rng, 8, 36),
                    count=rng.choice([1, 1, 2, 4]), rule=rng.randint(0, 1), J=True, nsweeps=_log(rng, 20, 150),
                    EM=rng.random() < 0.8)
    if kind == "msc":
        dims = rng.choice([2, 3])
        Lx = 128 * rng.randint(1, 16) if dims == 2 else 128 * rng.randint(1, 2)
        Ly = _even(rng, 64, 4096) if dims == 2 else _even(rng, 16, 200)
        Lz = 1 if dims == 2 else _even(rng, 16, 200)
        n = max(1, min(rng.randint(1, 8), 60_000_000 // (Lx * Ly * Lz)))
        return dict(kind="msc", dims=dims, Lx=Lx, Ly=Ly, Lz=Lz, count=1, rule=rng.randint(0, 1), nsweeps=n,
                    EM=rng.random() < 0.7)
    if kind == "sg":
        L = 16 * rng.randint(1, 3)
        count = _log(rng, 2, 64)
        n = max(1, min(rng.randint(5, 40), 42_000_000 // (L ** 3 * count)))
        return dict(kind="sg", dims=3, Lx=L, Ly=L, Lz=L, count=count, rule=rng.randint(0, 1), nsweeps=n,
                    EM=rng.random() < 0.7)
    if kind == "dcb":
        tile = rng.choice([64, 128, 128, 256])
        L = 2 * tile * _log(rng, 1, 4096 // (2 * tile))
        count, hits = rng.randint(1, 3), rng.choice([1, 2, 5, 10, 30])
        n = max(1, min(rng.randint(1, 20), 2_400_000_000 // (L * L * count * hits)))
        return dict(kind="dcb", L=L, count=count, tile=tile, hits=hits, nsweeps=n)
    if kind == "pa":
        Ls = sorted(rng.sample([8, 16, 32, 64, 128], rng.randint(1, 3)))
        R = _log(rng, 1000, 16384)
        c = {"L%d" % i: L for i, L in enumerate(Ls)}
        return dict(kind="pa", R=R, theta=rng.randint(3, 10), nsteps=rng.randint(3, 8), **c)
    if kind == "pt":
        return dict(kind="pt", L=rng.choice([16, 32, 64, 128]), n_temps=rng.randint(8, 32),
                    n_sets=_log(rng, 4, 64), theta=rng.randint(2, 10), rounds=rng.randint(3, 10))
    if kind == "muca":
        L = rng.choice([16, 24, 32, 48, 64, 96, 128])
        return dict(kind="muca", L=L, walkers=_log(rng, 500, 16384), nsweeps=max(1, 16384 // (L * L)),
                    record=rng.random() < 0.7)
    L = rng.choice([16, 32, 64])
    nwin = {16: 4, 32: 16, 64: 64}[L]
    return dict(kind="wl", L=L, nwin=nwin, walkers=64 * rng.randint(1, 4), nsweeps=rng.randint(1, max(1, 8192 // (L * L))))


# -------------------------------------------------------------- equilibrium data
def _entropy(L):
    """ln g(E) of the L x L torus at the levels E = 4 k - 2 N, k = 0 .. N / 2, up
    to a constant, from the infinite lattice's exact internal energy u(beta)
    (dS/dE = beta): weights as a converged multicanonical run holds them."""
    N = L * L
    b = np.linspace(1e-4, 2.5, 20001)
    kappa = 2.0 * np.sinh(2 * b) / np.cosh(2 * b) ** 2
    x, y = np.ones_like(b), np.sqrt(np.maximum(1.0 - kappa ** 2, 1e-14))
    for _ in range(12):  # arithmetic-geometric mean: K = pi / (2 agm)
        x, y = 0.5 * (x + y), np.sqrt(x * y)
    K = math.pi / (2.0 * x)
    u = -(1.0 / np.tanh(2 * b)) * (1.0 + (2.0 / math.pi) * (2.0 * np.tanh(2 * b) ** 2 - 1.0) * K)
    e = (4.0 * np.arange(N // 2 + 1) - 2.0 * N) / N
    beta = np.interp(-e, -u, b)  # -u grows with beta
    s = np.concatenate([[0.0], np.cumsum(0.5 * (beta[1:] + beta[:-1]) * 4.0)])
    return s - s[-1]


def _windows(L, nwin, overlap=8):
    """nwin windows of equal width over the levels 0 .. N / 2, neighbours sharing
    `overlap` levels."""
    K = L * L // 2
    width = -(-(K + 1 + (nwin - 1) * overlap) // nwin)
    lo = [min(i * (width - overlap), K - width + 1) for i in range(nwin)]
    hi = [v + width - 1 for v in lo]
    hi[-1] = K
    return lo, hi


# ------------------------------------------------------------------- prepare
def prepare(case, seed):
    kind = case["kind"]
    ctx = mcs.Context(0)
    st = dict(case=case, ctx=ctx, seed=1000 + seed, sweep0=0)
    if kind in ("sweep", "msc", "sg"):
        shape = (case["Lx"], case["Ly"]) + ((case["Lz"],) if case["dims"] == 3 else ())
        layout = mcs.INT8 if kind == "sweep" else mcs.MSC64
        g = mcs.make_geom(case["dims"], shape, layout=layout, count=case["count"])
        lat = mcs.lattice_tensor(g, DEV)
        ctx.init(g, lat, mcs.HOT, st["seed"], 0)
        st.update(g=g, lat=lat, J=None, ws=None, EM=None)
        if kind == "sg":
            st["J"] = torch.empty((g.count, g.dims * g.N), dtype=torch.int64, device=DEV)
            ctx.couplings_msc64(g, st["J"], st["seed"], 0)
            st["beta"] = 1.0
        elif case.get("J"):
            st["J"] = torch.empty(g.dims * g.N, dtype=torch.int8, device=DEV)
            ctx.couplings(g, st["J"], st["seed"])
            st["beta"] = 1.0
        else:
            st["beta"] = BETA_C if case["dims"] == 2 else BETA_C3
        # several int8 lattices run at temperatures around the critical one
        st["betas"] = [st["beta"] * (0.9 + 0.2 * i / max(1, g.count - 1)) for i in range(g.count)]
        if kind == "sweep":
            nb = ctx.sweep_workspace_bytes(g)
            st["ws"] = torch.empty(nb, dtype=torch.uint8, device=DEV) if nb else None
        if case["EM"]:
            st["EM"] = torch.zeros((case["nsweeps"], g.count * g.lanes, 2), dtype=torch.int64, device=DEV)
    elif kind == "dcb":
        g = mcs.make_geom(2, case["L"], count=case["count"])
        lat = mcs.lattice_tensor(g, DEV)
        ctx.init(g, lat, mcs.HOT, st["seed"], 0)
        st.update(g=g, lat=lat, ws=torch.empty(ctx.dcb_workspace_bytes(g), dtype=torch.uint8, device=DEV),
                  EM=torch.zeros((case["nsweeps"], g.count, 2), dtype=torch.int64, device=DEV))
    elif kind == "pa":
        Ls = [case["L%d" % i] for i in range(4) if "L%d" % i in case]
        beta = np.arange(case["nsteps"] + 1) / 200.0
        st.update(Ls=Ls, beta=beta, pops=ctx.pa_population_tensors(Ls, case["R"]),
                  ws=torch.empty(ctx.pa_workspace_bytes(Ls, case["R"], case["theta"], beta), dtype=torch.uint8,
                                 device=DEV))
    elif kind == "pt":
        n = case["n_temps"]
        beta = [0.35 + 0.2 * i / (n - 1) for i in range(n)]
        st.update(beta=beta, pt=ctx.pt_state(case["L"], n, case["n_sets"], st["seed"]),
                  ws=torch.empty(ctx.pt_workspace_bytes(case["L"], beta, case["n_sets"], case["theta"],
                                                        case["rounds"]), dtype=torch.uint8, device=DEV))
    elif kind == "muca":
        L, W = case["L"], case["walkers"]
        spins, E = ctx.muca_start(L, W, st["seed"], start=mcs.MUCA_STRATIFIED)
        st.update(spins=spins, E=E, lnW=-_entropy(L), ws=ctx.muca_workspace(L, W),
                  H=torch.zeros(L * L // 2 + 1, dtype=torch.int64, device=DEV))
    elif kind == "wl":
        L, M = case["L"], case["walkers"]
        lo, hi = _windows(L, case["nwin"])
        ws = ctx.wl_workspace(L, lo, hi, M)
        spins, E = ctx.win_drive(L, lo, hi, M, st["seed"], ws=ws)
        wmax = max(h - l for l, h in zip(lo, hi)) + 1
        S = _entropy(L)
        G = torch.zeros((len(lo), wmax), dtype=torch.int64)
        for i in range(len(lo)):
            w = np.round((S[lo[i]:hi[i] + 1] - S[lo[i]]) * 4294967296.0).astype(np.int64)
            G[i, :w.size] = torch.from_numpy(w)
        W = len(lo) * M
        st.update(lo=lo, hi=hi, ws=ws, spins=spins, E=E, G=G.repeat_interleave(M, 0).to(DEV),
                  H=torch.zeros((W, wmax), dtype=torch.int32, device=DEV),
                  flags=torch.zeros(W, dtype=torch.int32, device=DEV), inc=[1 << 22] * len(lo), act=[1] * len(lo))
    else:
        raise ValueError("unknown kind %r" % kind)
    return st


# ----------------------------------------------------------------------- run
def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["case"]["kind"]
    s0 = st["sweep0"]
    if kind == "sweep" and case["count"] > 1:
        ctx.sweep_betas(st["g"], st["lat"], st["betas"], st["seed"], case["nsweeps"], sweep0=s0, rule=case["rule"],
                        J=st["J"], EM=st["EM"], ws=st["ws"])
    elif kind in ("sweep", "msc"):
        ctx.sweep(st["g"], st["lat"], st["beta"], st["seed"], case["nsweeps"], sweep0=s0, rule=case["rule"],
                  J=st["J"], EM=st["EM"], ws=st["ws"])
    elif kind == "sg":
        ctx.sweep_sg_msc64(st["g"], st["lat"], st["J"], st["beta"], st["seed"], case["nsweeps"], sweep0=s0,
                           rule=case["rule"], EM=st["EM"])
    elif kind == "dcb":
        ctx.sweep_dcb(st["g"], st["lat"], BETA_C, st["seed"], case["nsweeps"], case["tile"], case["hits"], sweep0=s0,
                      EM=st["EM"], ws=st["ws"])
    elif kind == "pa":  # a fresh anneal each time, as for independent runs
        r = ctx.pa_anneal(st["Ls"], case["R"], case["theta"], st["seed"], st["beta"], st["pops"], ws=st["ws"])
        final = [p[:case["R"] * L * L] for p, L in zip(st["pops"], st["Ls"])]
        return dict(Ctot=r["Ctot"], lnQ=r["lnQ"], lnZ=r["lnZ"], hist=r["hist"], final=final)
    elif kind == "pt":
        E_at = ctx.pt_run(case["L"], st["beta"], case["theta"], st["seed"], st["pt"], s0, case["rounds"],
                          ws=st["ws"])
        st["sweep0"] = s0 + case["rounds"]
        p = st["pt"]
        return dict(E_at=E_at, spins=p["spins"], temp_of=p["temp_of"], replica_at=p["replica_at"],
                    accepted=p["accepted"])
    elif kind == "muca":
        ctx.muca_sweeps(case["L"], st["spins"], st["E"], st["lnW"], st["seed"], s0, case["nsweeps"], case["record"],
                        st["H"], st["ws"])
        st["sweep0"] = s0 + case["nsweeps"]
        return dict(spins=st["spins"], E=st["E"], H=st["H"])
    elif kind == "wl":
        ctx.wl_sweeps(case["L"], st["lo"], st["hi"], case["walkers"], st["inc"], st["act"], st["seed"], s0,
                      case["nsweeps"], st["spins"], st["E"], st["G"], st["H"], st["flags"], ws=st["ws"])
        st["sweep0"] = s0 + case["nsweeps"]
        return dict(spins=st["spins"], E=st["E"], G=st["G"], H=st["H"], flags=st["flags"])
    st["sweep0"] = s0 + case["nsweeps"]
    return dict(spins=st["lat"]) if st["EM"] is None else dict(spins=st["lat"], EM=st["EM"])


# ---------------------------------------------------------------------- work
# Integer operations per attempted update that the definition of the chains asks
# for.  Checkerboard updates draw one byte each, a sixteenth of a Philox block of
# ten rounds of two wide multiplies and four exclusive ors (60 operations), and
# share the bit-parallel rest; sequential walkers draw a whole word, a quarter of
# a block, and decide one site at a time (neighbours, table entry, test, count).
# Words of 64 realisations share one draw per site.
OPS_CHECKERBOARD = 60 / 16 + 1
OPS_SEQUENTIAL = 60 / 4 + 10


def work(case):
    kind = case["kind"]
    if kind in ("sweep", "msc", "sg"):
        N = case["Lx"] * case["Ly"] * (case["Lz"] if case["dims"] == 3 else 1)
        lanes = 1 if kind == "sweep" else 64
        site = 1 if kind == "sweep" else 8
        em = 16 * case["nsweeps"] * case["count"] * lanes if case["EM"] else 0
        nbytes = 2 * site * N * case["count"] + em
        if kind == "sg":
            nbytes += 8 * case["dims"] * N * case["count"]
        elif case.get("J"):
            nbytes += case["dims"] * N
        ops = OPS_CHECKERBOARD if kind != "sg" else 60 / 16 / 64 + 1
        return dict(bytes=nbytes, flops=ops * N * lanes * case["count"] * case["nsweeps"])
    if kind == "dcb":
        n = case["L"] ** 2 * case["count"]
        return dict(bytes=2 * n + 16 * case["nsweeps"] * case["count"],
                    flops=OPS_CHECKERBOARD * n * case["hits"] * case["nsweeps"])
    if kind == "pa":
        n = sum(case["L%d" % i] ** 2 for i in range(4) if "L%d" % i in case)
        return dict(bytes=n * case["R"], flops=OPS_CHECKERBOARD * n * case["R"] * case["theta"] * case["nsteps"])
    if kind == "pt":
        n = case["L"] ** 2 * case["n_temps"] * case["n_sets"]
        return dict(bytes=2 * n, flops=OPS_CHECKERBOARD * n * case["theta"] * case["rounds"])
    if kind == "muca":
        n = case["L"] ** 2 * case["walkers"]
        return dict(bytes=2 * n, flops=OPS_SEQUENTIAL * n * case["nsweeps"])
    lo, hi = _windows(case["L"], case["nwin"])
    W = case["nwin"] * case["walkers"]
    wide = max(h - l for l, h in zip(lo, hi)) + 1
    return dict(bytes=2 * W * (case["L"] ** 2 + 12 * wide), flops=OPS_SEQUENTIAL * W * case["L"] ** 2 * case["nsweeps"])


def exact(case, seed):
    """None: the outputs are whole numbers of a random process (spins, energies,
    counts), equal bit for bit or not; the annealing's weights sums follow from
    its populations and have no value of their own without the whole chain."""
    return None
