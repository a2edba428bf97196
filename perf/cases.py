"""Workloads of the library as its users run them, for timing and for checking.

Every case is one or several whole population-annealing runs through the
public entry points (`pa_run`, `pa_run_batch`, `Server`).  A case is a dict:

  entry      "run" (one pa_run), "batch" (one pa_run_batch of `n` runs) or
             "serve" (`n` requests submitted to a running server)
  L, q, R    lattice side, states, target population (the first run's)
  theta      sweeps per temperature step
  steps      temperature steps (K - 1)
  beta0, beta1   the inverse temperatures run from beta0 to beta1 in equal steps
  n_beta     if set: the piecewise protocol of Tables I-III instead
  poisson    Poisson resampling (else multinomial)
  ground     ground-state start (a heating run; beta1 < beta0)
  hist, mag, widths, final   the outputs asked for
  mixed      runs of several lattice sides, q and populations (as
             `workloads.mixed_runs` and `workloads.serving_requests` mix them)
"""
import math

import numpy as np
import torch

import paper_1704_01888_amd as pa
from paper_1704_01888_amd import workloads

DEFAULTS = dict(entry="run", n=1, L=32, q=10, R=1000, theta=10, steps=20, beta0=0.0, beta1=1.6, n_beta=0,
                poisson=True, ground=False, hist=False, mag=False, widths=False, final=False, mixed=False)


def _case(name, **kw):
    return dict(DEFAULTS, name=name, **kw)


def listed():
    return [
        # The smallest run: one 8x8 anneal of 1000 replicas, 200 short steps,
        # where launches and latency count (the benchmark's small run).
        _case("small_8", L=8, q=8, R=1000, steps=200, poisson=False),
        # Averages over independent seeds: 20 of the same in one batch.
        _case("batch_8", entry="batch", n=20, L=8, q=8, R=1000, steps=200, poisson=False),
        # An ordinary cooling run with energy histograms (the benchmark's
        # 32x32 workload with fewer steps).
        _case("cool_32", L=32, q=10, R=20000, steps=40, hist=True),
        # A heating run from ground states through the transition (hysteresis
        # curves), with every observable and the final population.
        _case("heat_32", L=32, q=6, R=10000, steps=60, beta0=1.6, beta1=1.0, poisson=False, ground=True, hist=True,
              mag=True, widths=True, final=True),
        # Rows of Tables II and III: few replicas, many sweeps, the widths of
        # the energy and magnetisation histograms.
        _case("tables_64", entry="batch", n=4, L=64, q=8, R=1000, theta=100, steps=0, n_beta=100, mag=True,
              widths=True),
        # The largest population in memory: the first steps of the benchmark's
        # headline run.
        _case("large_128", L=128, q=10, R=200000, theta=20, steps=3, beta1=0.0096),
        # Very many small lattices: precise free energies of a small system.
        _case("many_16", L=16, q=10, R=1000000, steps=10, beta1=0.1, hist=True),
        # A side that is not a multiple of 4, ragged population.
        _case("side_50", L=50, q=5, R=3001, steps=20, beta1=1.2),
        # A side that is a multiple of 4 without a power of two, q of Table I's
        # largest value.
        _case("side_100", L=100, q=20, R=5003, steps=20, beta1=1.7, mag=True),
        # A campaign over lattice sides, q and populations in one batch.
        _case("mixed_batch", entry="batch", n=6, R=10000, steps=12, beta1=1.2, mixed=True),
        # Lattices beyond one workgroup's LDS.
        _case("side_1024", L=1024, q=10, R=96, steps=5, beta1=1.0),
        # Requests of mixed sizes answered by the serving loop.
        _case("serve_mix", entry="serve", n=12, R=2000, steps=40, beta1=1.2, mixed=True),
    ]


MOST_ATTEMPTS = 1.2e11   # site updates of a drawn case (large_128 has 2e11)


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "heat", "batch", "mixed", "serve", "tiled"])
    c = dict(DEFAULTS)
    c["q"] = _log(rng, 2, 24)
    c["theta"] = _log(rng, 2, 100)
    c["steps"] = _log(rng, 3, 100)
    c["poisson"] = rng.random() < 0.7
    c["beta1"] = round(min(0.02 * c["steps"], 1.6), 4)
    if kind == "tiled":
        c["L"] = 4 * rng.randint(65, 300) if rng.random() < 0.5 else rng.choice([512, 1024, 2048])
        c["R"] = _log(rng, 16, 200)
        c["steps"] = rng.randint(2, 6)
        c["theta"] = _log(rng, 2, 20)
    elif kind in ("run", "heat", "batch"):
        c["L"] = 2 * rng.randint(4, 64) if rng.random() < 0.4 else rng.choice([8, 16, 24, 32, 48, 64, 96, 128])
        c["R"] = _log(rng, 100, 1000000 if kind == "run" else 20000)
        for o in ("hist", "mag", "widths"):
            c[o] = rng.random() < 0.3
        if kind == "heat":
            c["ground"], c["beta0"] = True, 1.6
            c["final"] = not c["poisson"] and c["L"] * c["L"] * c["R"] < 2e7   # sizes that do not depend on the seed
            c["beta1"] = round(max(1.6 - 0.01 * c["steps"], 0.9), 4)
        if kind == "batch":
            c["entry"], c["n"] = "batch", rng.randint(2, 24)
    else:
        c["entry"] = "batch" if kind == "mixed" else "serve"
        c["mixed"], c["n"], c["R"] = True, rng.randint(2, 12), _log(rng, 300, 10000)
    # fewer steps, then sweeps, then replicas, until the case is small enough
    while _attempts(c) > MOST_ATTEMPTS:
        if c["steps"] > 4:
            c["steps"] //= 2
        elif c["theta"] > 4:
            c["theta"] //= 2
        else:
            c["R"] = max(1, c["R"] // 2)
    return c


def _runs(case, seed):
    """The run descriptions of a case (dicts of Desc fields)."""
    if case["n_beta"]:
        beta = workloads.table_betas(case["q"], case["n_beta"])
    else:
        n, b0, b1 = case["steps"], case["beta0"], case["beta1"]
        beta = np.array([b0 + (b1 - b0) * i / n for i in range(n + 1)])
    outputs = ((pa.OUT_HIST if case["hist"] else 0) | (pa.OUT_MAG if case["mag"] else 0) |
               (pa.OUT_WIDTHS if case["widths"] else 0) | (pa.OUT_FINAL if case["final"] else 0))
    runs = []
    for r in range(case["n"]):
        L, q, R = case["L"], case["q"], case["R"]
        if case["mixed"]:
            sides = [16, 24, 32, 48, 64] if case["entry"] == "batch" else [16, 32, 64, 128]
            L = sides[(3 * r + 1) % len(sides)]
            q = [5, 6, 8, 10, 20][(2 * r) % 5]
            R = int(case["R"] * [1.0, 5.3, 0.51, 2.7][r % 4]) + r
        runs.append(dict(L=L, q=q, R=R, beta=beta, theta=case["theta"], seed=7919 * seed + 101 * r + 1,
                         resample=pa.RESAMPLE_POISSON if case["poisson"] else pa.RESAMPLE_MULTINOMIAL,
                         init=pa.INIT_GROUND if case["ground"] else pa.INIT_RANDOM, outputs=outputs))
    return runs


def _attempts(case):
    return sum(float(r["L"]) ** 2 * r["R"] * r["theta"] * (len(r["beta"]) - 1) for r in _runs(case, 0))


_context = []


def prepare(case, seed):
    descs = [pa.Desc(**r) for r in _runs(case, seed)]
    if case["entry"] == "serve":
        # a server of its own, as a serving program keeps one running
        ctx = pa.Context(0)
        arena = sum(int(pa.pa_plan(d).workspace_bytes) for d in descs)
        return dict(entry="serve", descs=descs, server=pa.Server(ctx, arena, max_slots=16))
    if not _context:
        _context.append(pa.Context(0))
    need = pa.pa_plan_batch(descs) if case["entry"] == "batch" else int(pa.pa_plan(descs[0]).workspace_bytes)
    return dict(entry=case["entry"], descs=descs, ctx=_context[0],
                ws=torch.empty(need, dtype=torch.uint8, device="cuda:0"))


# Everything a run returns but the launch counts and profiling times.
_SKIP = ("kernel_ms", "kernel_launches")


def _together(results):
    """One array per output: the runs' arrays one after another."""
    keys = [k for k in results[0] if k not in _SKIP]
    if len(results) == 1:
        return {k: results[0][k] for k in keys}
    return {k: np.concatenate([r[k].reshape(-1) for r in results]) for k in keys}


def run(state):
    if state["entry"] == "run":
        return _together([pa.pa_run(state["ctx"], state["descs"][0], workspace=state["ws"])])
    if state["entry"] == "batch":
        return _together(pa.pa_run_batch(state["ctx"], state["descs"], workspace=state["ws"]))
    server = state["server"]
    tickets = [server.submit(d) for d in state["descs"]]
    return _together([server.wait(t)[0] for t in tickets])


def work(case):
    """Bytes: every step reads each new replica's ancestor and writes the
    replica (one byte per site), once each; the histograms are written.  Ops:
    40 32-bit integer operations per site update (half a Philox4x32-10 block,
    the proposal, eight neighbour comparisons, the acceptance test)."""
    moved = flops = 0.0
    for r in _runs(case, 0):
        sites, steps = float(r["L"]) ** 2 * r["R"], len(r["beta"]) - 1
        moved += 2.0 * sites * steps + sites
        flops += 40.0 * sites * r["theta"] * steps
        if case["hist"]:
            moved += 8.0 * r["L"] ** 2 * (steps + 1)
    return {"bytes": moved, "flops": flops}


# ---------------------------------------------------------------------------
# The same runs in plain 64-bit torch and numpy: population annealing as
# arXiv:1704.01888 Sec. 2 states it, with the conventions of include/pa.h
# (Philox4x32-10 counters, integer thresholds and weights, ancestor order).
# ---------------------------------------------------------------------------
_M32 = 0xFFFFFFFF
INIT, SWEEP, RESAMPLE, PLAN, GROUND = 0, 1, 2, 3, 4


def _hi(p):
    return (p >> 32) & _M32


def _philox(c0, c1, c2, c3, seed):
    """Four 32-bit words per counter (int64 tensors and Python ints mix)."""
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2
        c0, c1, c2, c3 = _hi(p1) ^ c1 ^ k0, p1 & _M32, _hi(p0) ^ c3 ^ k1, p0 & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1, c2, c3


def _mulhi64(x1, x0, s):
    """floor(x s / 2^64) for x = x1 2^32 + x0 (tensors) and 0 <= s < 2^63."""
    s1, s0 = s >> 32, s & _M32
    lo, a, b = x0 * s0, x0 * s1, x1 * s0
    mid = _hi(lo) + (a & _M32) + (b & _M32)
    return x1 * s1 + _hi(a) + _hi(b) + (mid >> 32)


def _schedule(run):
    """Population sizes R_i (Poisson by inversion from the mode outwards)."""
    out = [run["R"]] * len(run["beta"])
    if run["resample"] != pa.RESAMPLE_POISSON:
        return out
    lam = float(run["R"])
    for i in range(1, len(out)):
        w = _philox(0, 0, i, PLAN << 28, run["seed"])
        u = float(((w[1] << 32) | w[0]) >> 11) * 2.0 ** -53
        m = math.floor(lam)
        acc = hi_p = lo_p = math.exp(-lam + m * math.log(lam) - math.lgamma(m + 1.0))
        hi = lo = n = m
        while u >= acc:
            hi += 1
            hi_p = hi_p * lam / hi
            acc, n = acc + hi_p, hi
            if u < acc:
                break
            if lo > 0:
                lo_p = lo_p * lo / lam
                lo -= 1
                acc, n = acc + lo_p, lo
        out[i] = n
    return out


def _energy(s):
    return -((s == s.roll(-1, 2)).sum((1, 2)) + (s == s.roll(-1, 1)).sum((1, 2)))


def _half_sweep(s, colour, i, t, beta, run):
    """One colour of one sweep of every replica (s: [R][L][L] int64)."""
    R, L = s.shape[0], s.shape[1]
    q, dev = run["q"], s.device
    m = torch.arange(L * L // 4, device=dev)
    k = torch.arange(R, device=dev)[:, None]
    w = _philox(m[None, :], k, i, (SWEEP << 28) | (t << 1) | colour, run["seed"])
    prop = torch.stack((w[0], w[2]), 2).reshape(R, L, L // 2)
    acc = torch.stack((w[1], w[3]), 2).reshape(R, L, L // 2)
    y = torch.arange(L, device=dev)[:, None]
    x = 2 * torch.arange(L // 2, device=dev)[None, :] + ((y + colour) & 1)
    cur = s[:, y, x]
    r = _hi(prop * (q - 1))
    new = r + (r >= cur)
    dE = torch.zeros_like(cur)
    for ny, nx in ((y, (x + 1) % L), (y, (x - 1) % L), ((y + 1) % L, x), ((y - 1) % L, x)):
        nb = s[:, ny, nx]
        dE += (nb == cur).long() - (nb == new).long()
    T = torch.tensor([1 << 32] * 5 + [int(math.floor(math.ldexp(math.exp(-beta * d), 32))) for d in (1, 2, 3, 4)],
                     device=dev)
    s[:, y, x] = torch.where(acc < T[dE + 4], new, cur)


def _fwhm(h, nb):
    """Width at half maximum of the piecewise-linear curve through the counts."""
    H = int(h.max())
    if H == 0:
        return 0.0
    at = np.nonzero(2 * h >= H)[0]
    jl, jr = int(at[0]), int(at[-1])
    half = 0.5 * H
    l0, r1 = (float(h[jl - 1]) if jl else 0.0), (float(h[jr + 1]) if jr + 1 < nb else 0.0)
    return (jr + (float(h[jr]) - half) / (float(h[jr]) - r1)) - (jl - 1 + (half - l0) / (float(h[jl]) - l0))


def _exact_run(run, case):
    dev = "cuda:0" if torch.cuda.is_available() else "cpu"
    L, q, beta, seed = run["L"], run["q"], [float(b) for b in run["beta"]], run["seed"]
    N, K, R_i = L * L, len(beta), _schedule(run)
    Kb = 63 - (max(R_i) - 1).bit_length()
    k = torch.arange(run["R"], device=dev)[:, None]
    if run["init"] == pa.INIT_GROUND:
        w = _philox(0, k, 0, GROUND << 28, seed)
        s = _hi(w[0] * q).expand(-1, N).reshape(-1, L, L).clone()
    else:
        w = _philox(torch.arange(N // 4, device=dev)[None, :], k, 0, INIT << 28, seed)
        s = _hi(torch.stack(w, 2).reshape(-1, L, L) * q)
    out = {f: [] for f in ("E_sum", "E_mean", "lnQ", "minus_beta_F", "hist", "Mt_sum", "M_mean", "mhist", "width_e",
                           "width_m")}
    F = math.log(q) + 2.0 * N * beta[0] if run["init"] == pa.INIT_GROUND else N * math.log(q)
    lnq, anc = 0.0, torch.arange(run["R"], device=dev)
    for i in range(K):
        if i:
            db = beta[i] - beta[i - 1]
            ref = int(E.min() if db >= 0 else E.max())
            d = (E - ref).abs()
            W = [int(round(math.ldexp(math.exp(-abs(db) * x), Kb))) for x in range(int(d.max()) + 1)]
            h = torch.bincount(d).tolist()
            lnq = -db * ref + math.log(math.fsum(n * math.exp(-abs(db) * x) for x, n in enumerate(h))) - \
                math.log(R_i[i - 1])
            F += lnq
            C = torch.tensor(W, device=dev)[d].cumsum(0)
            w = _philox(torch.arange(R_i[i], device=dev), 0, i, RESAMPLE << 28, seed)
            u = _mulhi64(w[1], w[0], int(C[-1]))
            anc = torch.searchsorted(C, u, right=True).sort().values
            s = s[anc]
            for t in range(run["theta"]):
                for colour in (0, 1):
                    _half_sweep(s, colour, i, t, beta[i], run)
        E = _energy(s)
        h = torch.bincount(E + 2 * N, minlength=2 * N + 1).cpu().numpy()
        M = torch.stack([(s == a).sum((1, 2)) for a in range(q)]).amax(0)
        hm = torch.bincount(M, minlength=N + 1).cpu().numpy()
        Es, Ms, R = int(E.sum()), int(M.sum()), R_i[i]
        for f, v in (("E_sum", Es), ("E_mean", Es / R), ("lnQ", lnq), ("minus_beta_F", F), ("hist", h), ("mhist", hm),
                     ("Mt_sum", Ms), ("M_mean", (q * Ms - N * R) / ((q - 1) * R)), ("width_e", _fwhm(h, 2 * N + 1) / N),
                     ("width_m", _fwhm(hm, N + 1) * q / ((q - 1) * N))):
            out[f].append(v)
    keys = ["E_sum", "E_mean", "lnQ", "minus_beta_F"]
    keys += (["hist"] if case["hist"] else []) + (["Mt_sum", "M_mean"] if case["mag"] else [])
    keys += (["mhist"] if case["mag"] and case["hist"] else []) + (["width_e"] if case["widths"] else [])
    keys += ["width_m"] if case["mag"] and case["widths"] else []
    types = dict(E_sum=np.int64, Mt_sum=np.int64, hist=np.uint32, mhist=np.uint32)
    res = {f: np.array(out[f], dtype=types.get(f, np.float64)) for f in keys}
    res["R_i"] = np.array(R_i, np.uint64)
    if case["final"]:
        res["final_spins"] = s.reshape(-1, N).to(torch.uint8).cpu().numpy()
        res["final_E"] = E.to(torch.int32).cpu().numpy()
        res["last_anc"] = anc.cpu().numpy().astype(np.uint32)
    return res


def exact(case, seed):
    runs = _runs(case, seed)
    # one half-sweep costs about 1.2 ms of launches and 2 ns per Philox block
    cost = sum(2.0 * r["theta"] * (len(r["beta"]) - 1) * (1.2e-3 + 2e-9 * r["R"] * r["L"] ** 2 / 4) for r in runs)
    if cost > 12.0:
        return None
    return _together([_exact_run(r, case) for r in runs])
