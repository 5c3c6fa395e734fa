"""The work that users of this framework have it do, as cases that can be timed and compared.

Three kinds of case, each through the public binding (`paper_1006_0252_amd.pa`, `.learned`):
  anneal   initialise a run or a batch of runs and take it through a window of a schedule: resample,
           sweep and measure at every temperature (eagerly or as one captured graph);
  train    one full-batch training step of the network that proposes temperature steps;
  averages the weighted averages of an ensemble and their bootstrap errors.

listed() names the cases, draw() gives further ones of the same ranges.  An anneal starts from the
seeds every time, so a pass can be repeated; it hands back every run's records and the final energies
and spins of its replicas.  A population's size fluctuates about its target R0 by about sqrt(R0) and
stays on the device, so the replicas handed back are those that every run is sure to have (R0 less
ten standard deviations, whole groups of 64).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1006_0252_amd import learned, pa

DEV = "cuda:0"


def _anneal(name, dim, L, R0, n_runs, layout, couplings, beta0, dbeta, n_steps, n_sweeps, pairs=False, graph=False,
            L_last=0, R_last=0):
    """L_last, R_last > 0: the batch's realisations take sides L, L + 2, .. L_last and target sizes
    between R0 and R_last (four runs of a realisation each)."""
    return dict(name=name, kind="anneal", dim=dim, L=L, R0=R0, n_runs=n_runs, layout=layout, couplings=couplings,
                beta0=beta0, dbeta=dbeta, n_steps=n_steps, n_sweeps=n_sweeps, pairs=pairs, graph=graph, L_last=L_last,
                R_last=R_last)


def listed():
    return [
        # one small run stepped by hand, a whole schedule: launches and latency are all there is
        _anneal("ring_single", 1, 64, 1000, 1, "u8", "pm1", 0.0, 0.1, 50, 5),
        # the 1D bias measurement: 200 runs of a realisation, the whole schedule one graph
        _anneal("ring_ensemble", 1, 64, 1000, 200, "u8", "pm1", 0.0, 0.1, 50, 5, graph=True),
        # an ordinary 3D run in the default layout (a byte per spin), from the start of its schedule
        _anneal("cube8_bytes", 3, 8, 50000, 1, "u8", "pm1", 0.0, 0.05, 10, 10),
        # the learned-schedule target, around its glassy temperatures
        _anneal("cube12", 3, 12, 200000, 1, "bits64", "pm1", 0.9, 0.025, 6, 10),
        # the throughput configuration: the largest single population, first steps of its schedule
        _anneal("cube16_million", 3, 16, 1_000_000, 1, "bits64", "pm1", 0.0, 5.0 / 300, 3, 10),
        # many realisations of uneven size at once, with overlaps, one graph
        _anneal("batch_mixed", 3, 6, 10000, 256, "bits64", "pm1", 1.0, 0.05, 5, 10, True, True, 10, 100000),
        # a large cube deep in the cold phase, where only ties and free flips are accepted
        _anneal("cube20_cold", 3, 20, 20000, 1, "bits64", "pm1", 3.0, 0.05, 4, 10),
        # the paper's 3D ensemble: Gaussian couplings, 126 runs in pairs
        _anneal("gauss_cube8", 3, 8, 2000, 126, "u8", "gauss", 0.5, 0.02, 8, 100, True),
        # the same model on a smaller, odd-shaped cube
        _anneal("gauss_cube6", 3, 6, 2000, 8, "u8", "gauss", 0.8, 0.05, 2, 20, True),
        # the paper's 1D ensemble: Gaussian chain
        _anneal("gauss_chain", 1, 256, 1000, 200, "u8", "gauss", 0.0, 0.05, 20, 50, False, True),
        # a training step on the traces of the ring and the L = 8 cube
        dict(name="train_step", kind="train", B=10160),
        # errors of an 18-realisation ensemble
        dict(name="ensemble_errors", kind="averages", n_sets=18, M=200, n_obs=2, n_boot=200),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ring", "cube", "cube", "batch", "large", "gauss_cube", "gauss_chain", "train", "averages"])
    if kind == "train":
        return dict(kind="train", B=_log_int(rng, 300, 20000))
    if kind == "averages":
        return dict(kind="averages", n_sets=rng.randint(1, 25), M=2 * _log_int(rng, 10, 125), n_obs=rng.randint(1, 3),
                    n_boot=_log_int(rng, 50, 400))
    b0, db = rng.choice([0.0, 0.5, 1.0, 2.0, 3.0]), rng.uniform(0.01, 0.05)
    lay = rng.choice(["u8", "bits64"])
    if kind == "ring":
        n = rng.choice([1, _log_int(rng, 2, 200)])
        c = _anneal("", 1, 2 * _log_int(rng, 8, 512), _log_int(rng, 500, 5000), n, lay, "pm1", b0, db,
                    rng.randint(5, 30), rng.randint(2, 20), False, n > 1 and rng.random() < 0.5)
    elif kind == "cube":
        L = rng.choice([4, 6, 8, 10, 12, 14, 16])
        c = _anneal("", 3, L, min(_log_int(rng, 2000, 300000), 10 ** 9 // L ** 3), 1, lay, "pm1", b0, db,
                    rng.randint(2, 8), rng.randint(3, 10))
    elif kind == "batch":
        L = rng.choice([4, 6, 8, 10])
        c = _anneal("", 3, L, _log_int(rng, 2000, 20000), 4 * _log_int(rng, 1, 24), lay, "pm1", b0, db, rng.randint(2, 5),
                    rng.randint(5, 10), rng.random() < 0.5, rng.random() < 0.5, min(L + 2 * rng.randint(0, 2), 12),
                    _log_int(rng, 20000, 60000))
    elif kind == "large":
        L = rng.choice([18, 20, 24])
        c = _anneal("", 3, L, _log_int(rng, 2000, 20000), 1, lay, "pm1", b0, db, rng.randint(2, 4), rng.randint(3, 10))
    elif kind == "gauss_cube":
        L = rng.choice([4, 6, 8, 10])
        tabled = L in (4, 8)
        n = 2 * (_log_int(rng, 1, 40) if tabled else rng.randint(1, 4 if L < 10 else 2))
        c = _anneal("", 3, L, _log_int(rng, 500, 4000 if tabled else 2000), n, "u8", "gauss", max(b0, 0.4), db,
                    rng.randint(2, 4) if tabled else 1, rng.randint(10, 50 if tabled else 20), rng.random() < 0.5)
    else:
        n = _log_int(rng, 2, 200)
        c = _anneal("", 1, 16 * _log_int(rng, 2, 32), _log_int(rng, 500, 2000), n, "u8", "gauss", b0, db,
                    rng.randint(4, 12), rng.randint(10, 50), False, rng.random() < 0.5)
    del c["name"]
    return c


# ------------------------------------------------------------------ what an anneal consists of
def _betas(c):
    return np.array([c["beta0"] + c["dbeta"] * k for k in range(c["n_steps"] + 1)])


def _specs(c, seed):
    g = np.random.default_rng(3)  # sizes are the case's, whatever the seed
    specs = []
    for r in range(c["n_runs"]):
        L, R0, ds = c["L"], c["R0"], 7919 * seed + 1
        if c["L_last"]:
            if r % 4 == 0:
                L_real = int(g.choice(np.arange(c["L"], c["L_last"] + 1, 2)))
            L, ds = L_real, ds + r // 4
            R0 = int(g.integers(min(R0, c["R_last"]), max(R0, c["R_last"]) + 1))
        specs.append(dict(dim=c["dim"], L=L, R0=R0, seed=100_003 * seed + r + 1, disorder_seed=ds,
                          couplings=c["couplings"]))
    return specs


def _sure(R0):
    """Replicas that a population of target R0 is sure to have: whole groups of 64."""
    return max(64, int(R0 - 10 * math.sqrt(R0)) // 64 * 64)


def _views(run, c):
    """A run's records and, of its final buffers, the energies and spins of its first replicas."""
    m, cur = _sure(run.R0), c["n_steps"] % 2
    e_dtype, e_size = (torch.float64, 8) if c["couplings"] == "gauss" else (torch.int32, 4)
    row = int(run.sizes.spins_bytes) // run.capacity  # bytes of a replica in either layout
    return (run.record[: 128 * run.n_records].view(torch.float64).view(run.n_records, 16),
            run.energy[cur][: e_size * m].view(e_dtype), run.spins[cur][: row * m])


def prepare(case, seed):
    c = case
    if c["kind"] == "anneal":
        specs = _specs(c, seed)
        if c["n_runs"] == 1:
            s = specs[0]
            obj = pa.Run(s["dim"], s["L"], s["R0"], s["seed"], s["disorder_seed"], c["n_steps"] + 1,
                         layout=c["layout"], device=DEV, couplings=s["couplings"])
            runs = [obj]
        else:
            obj = pa.Batch(specs, c["n_steps"] + 1, layout=c["layout"], device=DEV)
            runs = obj.runs
        sched = pa.Schedule(_betas(c), c["n_sweeps"], max(r.n_bins for r in runs), device=DEV)
        graph = None
        if c["graph"]:
            obj.init()
            graph = obj.capture(sched, range(1, c["n_steps"] + 1), pairs=c["pairs"])
        return dict(case=c, obj=obj, sched=sched, graph=graph, views=[list(v) for v in zip(*(_views(r, c) for r in runs))])
    g = np.random.default_rng(1_000_003 * seed + 17)
    if c["kind"] == "train":
        x, target = _train_inputs(c, seed)
        net = learned.Network(learned.glorot_theta(seed), device=DEV)
        return dict(case=c, net=net, x=torch.from_numpy(x).to(DEV), target=torch.from_numpy(target).to(DEV))
    x, A, idx = _average_inputs(c, g)
    dev = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    n_out = c["n_obs"] + 3
    return dict(case=c, x=dev(x), A=dev(A), idx=dev(idx),
                out=torch.zeros((c["n_sets"], n_out), dtype=torch.float64, device=DEV),
                rep=torch.zeros((c["n_sets"], c["n_boot"], n_out), dtype=torch.float64, device=DEV),
                err=torch.zeros((c["n_sets"], n_out), dtype=torch.float64, device=DEV))


def run(state):
    c = state["case"]
    if c["kind"] == "train":
        net = state["net"]
        loss, grad = net.gradient(state["x"], state["target"])
        net.adam(3e-3)
        return dict(loss=loss, grad=grad, theta=net.theta)
    if c["kind"] == "averages":
        L, s = pa.lib(), torch.cuda.current_stream(DEV).cuda_stream
        x, A, out, rep, err = (state[k].data_ptr() for k in ("x", "A", "out", "rep", "err"))
        pa.check(L.pa_weighted_average_dev(c["n_sets"], c["M"], x, None, A, c["n_obs"], out, s), "averages")
        pa.check(L.pa_bootstrap_dev(c["n_sets"], c["M"], x, None, A, c["n_obs"], c["n_boot"],
                                    state["idx"].data_ptr(), rep, err, s), "bootstrap")
        return dict(out=state["out"], rep=state["rep"], err=state["err"])
    obj, sched = state["obj"], state["sched"]
    obj.init()
    if c["beta0"] > 0.0:
        obj.sweep(sched.start_sweeps())
    if state["graph"] is not None:
        state["graph"].launch()
    else:
        for k in range(1, c["n_steps"] + 1):
            if c["n_runs"] == 1:
                st = sched.step(k)
                obj.resample(st)
                obj.sweep(st)
                pa.measure([obj])
            else:
                obj.step(sched, k, pairs=c["pairs"])
    rec, energy, spins = state["views"]
    if c["n_runs"] == 1:
        return dict(records=rec[0], energy=energy[0], spins=spins[0])
    with torch.cuda.stream(obj.stream):
        return dict(records=torch.stack(rec), energy=torch.cat(energy), spins=torch.cat(spins))


def work(case):
    """Of an anneal: the attempts' draws, compares and flips (8 operations each: an eighth of a
    Philox call and the decision; 14 with a table of Gaussian thresholds), and each population read
    and written once per resample and once per call of sweeps."""
    c = case
    if c["kind"] == "train":
        return dict(bytes=c["B"] * 32 + 8833 * 26, flops=6 * c["B"] * 8640)
    if c["kind"] == "averages":
        n = c["n_sets"] * (c["n_boot"] + 1)
        return dict(bytes=8 * c["n_sets"] * c["M"] * (1 + c["n_obs"]) + 4 * c["n_boot"] * c["M"] + 8 * n * (c["n_obs"] + 3),
                    flops=n * c["M"] * (8 + 2 * c["n_obs"]))
    flops = nbytes = 0
    for s in _specs(c, 1):
        N = s["L"] if s["dim"] == 1 else s["L"] ** 3
        calls = c["n_steps"] + (1 if c["beta0"] > 0 else 0)
        flops += (14 if c["couplings"] == "gauss" else 8) * N * s["R0"] * c["n_sweeps"] * calls
        replica = (N if c["layout"] == "u8" else N / 8) + (8 if c["couplings"] == "gauss" else 4)
        nbytes += 2 * replica * s["R0"] * (calls + c["n_steps"])
    return dict(bytes=int(nbytes), flops=flops)


# ------------------------------------------------------------------ seeded inputs on the host
def _train_inputs(c, seed):
    """Feature rows (beta, ln N, ln R, E/N, var/N, skew) as traces of rings and cubes give them and
    step labels; every 50th row has no energy spread."""
    g = np.random.default_rng(1_000_003 * seed + 17)
    B = c["B"]
    x = np.empty((B, 6), np.float32)
    x[:, 0] = g.uniform(0.0, 5.0, B)
    x[:, 1] = np.log(g.choice([64.0, 512.0], B))
    x[:, 2] = g.choice([6.9, 10.8], B) + 0.02 * g.standard_normal(B)
    x[:, 3] = -1.7 * np.tanh(x[:, 0]) + 0.02 * g.standard_normal(B)
    x[:, 4] = 3.0 * np.exp(-1.2 * x[:, 0]) * np.exp(0.2 * g.standard_normal(B))
    x[:, 5] = 0.3 * g.standard_normal(B)
    x[::50, 4] = 0.0
    target = np.minimum(1.0, 0.3 / np.sqrt(np.exp(x[:, 1]) * np.maximum(x[:, 4], 1e-6)))
    return x, np.ascontiguousarray(target * np.exp(0.1 * g.standard_normal(B)), np.float64)


def _average_inputs(c, g):
    S, M = c["n_sets"], c["M"]
    x = 1147.0 + 0.6 * g.standard_normal((S, M))
    A = -224.0 + 0.5 * g.standard_normal((S, M, c["n_obs"]))
    return x, A, g.integers(0, M, (c["n_boot"], M)).astype(np.int32)


# ------------------------------------------------------------------ the same in plain numpy, 64 bits
def exact(case, seed):
    c = case
    if c["kind"] == "train":
        return _exact_train(c, seed)
    if c["kind"] == "averages":
        x, A, idx = _average_inputs(c, np.random.default_rng(1_000_003 * seed + 17))
        out = np.stack([_weighted(x[s], A[s]) for s in range(c["n_sets"])])
        rep = np.stack([[_weighted(x[s][i], A[s][i]) for i in idx] for s in range(c["n_sets"])])
        return dict(out=out, rep=rep, err=rep.std(axis=1, ddof=1))
    s = _specs(c, seed)[0]
    N = s["L"] if s["dim"] == 1 else s["L"] ** 3
    if c["n_runs"] > 1 or c["couplings"] != "pm1" or N * s["R0"] * c["n_sweeps"] * (c["n_steps"] + 1) > 4e7:
        return None  # minutes in numpy
    return dict(records=_exact_records(c, s, N), energy=None, spins=None)


def _weighted(x, A):
    w = np.exp(x - x.max())
    return np.concatenate([(w[:, None] * A).sum(0) / w.sum(), [x.max() + math.log(w.mean()), x.var(ddof=1), x.mean()]])


def _exact_train(c, seed):
    x, t = _train_inputs(c, seed)
    theta = learned.glorot_theta(seed)
    u = theta.view(np.uint32).astype(np.uint64)
    p = ((((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32)).view(np.float32).astype(np.float64)
    W1, b1 = p[:384].reshape(64, 6), p[384:448]
    W2, b2 = p[448:4544].reshape(64, 64), p[4544:4608]
    W3, b3 = p[4608:8704].reshape(64, 64), p[8704:8768]
    w4, b4 = p[8768:8832], p[8832]
    X, B = x.astype(np.float64), c["B"]
    X = np.stack([(X[:, 0] - 2.5) / 2.5, (X[:, 1] - 6) / 2, (X[:, 2] - 10) / 2.5, X[:, 3] + 1, X[:, 4] - 1, X[:, 5] / 2], 1)
    h1 = np.tanh(X @ W1.T + b1)
    h2 = np.tanh(h1 @ W2.T + b2)
    h3 = np.tanh(h2 @ W3.T + b3)
    z = h3 @ w4 + b4
    sp = np.maximum(z, 0) + np.log1p(np.exp(-np.abs(z)))
    var, ln_n = x[:, 4].astype(np.float64), x[:, 1].astype(np.float64)
    ok = var > 0
    err = np.where(ok, np.log(sp) - 0.5 * (ln_n + np.log(np.where(ok, var, 1.0))) - np.log(t), 0.0)
    gz = 2 / B * err / (1 + np.exp(-z)) / sp
    d3 = gz[:, None] * w4 * (1 - h3 * h3)
    d2 = (d3 @ W3) * (1 - h2 * h2)
    d1 = (d2 @ W2) * (1 - h1 * h1)
    grad = np.concatenate([(d1.T @ X).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0), (d3.T @ h2).ravel(), d3.sum(0),
                           gz @ h3, [gz.sum()]])
    step = 3e-3 * grad / (np.abs(grad) + 1e-8)  # Adam's first step: both moments are the gradient's own
    return dict(loss=np.array([(err * err).mean()]), grad=grad, theta=theta.astype(np.float64) - step)


# The counter-based draws make an anneal a function of its seeds: the generator, the rules of the
# checkerboard sweep and of the copy numbers, written out for whole arrays.
def _philox(c0, c1, c2, c3, seed):
    m32 = np.uint64(0xFFFFFFFF)
    c0, c1, c2, c3 = np.broadcast_arrays(*(np.asarray(v, np.uint64) for v in (c0, c1, c2, c3)))
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = c0 * np.uint64(0xD2511F53), c2 * np.uint64(0xCD9E8D57)
        c0, c1, c2, c3 = ((p1 >> np.uint64(32)) ^ c1 ^ np.uint64(k0), p1 & m32,
                          (p0 >> np.uint64(32)) ^ c3 ^ np.uint64(k1), p0 & m32)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack([c0, c1, c2, c3], axis=-1)


def _bits(words, n):
    """The first n stream bits of each row of calls [.., calls, 4]."""
    w = words.reshape(words.shape[:-2] + (-1,))
    b = (w[..., None] >> np.arange(32, dtype=np.uint64)) & np.uint64(1)
    return b.reshape(w.shape[:-1] + (-1,))[..., :n].astype(np.int64)


@functools.lru_cache(None)
def _ladder(m):
    """Inversion table of Poisson(2^m): floor(CDF 2^32), ending at the first n >= 2^m of mass below 2^-40."""
    lam, C, n = 2.0 ** m, [], 0
    p, F = math.exp(-lam), 0.0
    while True:
        F += p
        if n >= lam and p < 2.0 ** -40:
            return np.array(C + [1 << 32], np.uint64)
        C.append(min(int(math.floor(F * 2.0 ** 32)), 1 << 32))
        n += 1
        p = p * lam / n


def _copies(j, lam, k, seed, first):
    """Poisson(lam) copies of replica j at step k; first holds its first draws."""
    if not lam > 0:
        return 0
    q = int(math.ceil(lam / 64)) - 1 if lam > 64 else 0
    rem = lam - 64.0 * q
    f, e = math.frexp(rem)
    m = max(-20, e - 1 if f == 0.5 else e)
    keep = int(math.floor(math.ldexp(rem, 32 - m)))

    def draws(a, b):
        if b <= len(first):
            return first[a:b]
        return _philox(np.arange(a // 4, b // 4 + 1), j, k, 4, seed).ravel()[a % 4: a % 4 + b - a]

    n = int(np.searchsorted(_ladder(6), draws(0, q), side="right").sum()) if q else 0
    K = int(np.searchsorted(_ladder(m), draws(q, q + 1), side="right")[0])
    return n + int((draws(q + 1, q + 1 + K) < np.uint64(keep)).sum()) if K else n


def _exact_records(c, spec, N):
    dim, L, seed = spec["dim"], spec["L"], spec["seed"]
    i = np.arange(N)
    if dim == 1:
        nb, colour, z = np.stack([(i + 1) % N, (i - 1) % N]), i % 2, 2
    else:
        x, y, w = i % L, i // L % L, i // (L * L)
        at = lambda x, y, w: x % L + L * (y % L) + L * L * (w % L)  # noqa: E731
        nb = np.stack([at(x + 1, y, w), at(x, y + 1, w), at(x, y, w + 1), at(x - 1, y, w), at(x, y - 1, w), at(x, y, w - 1)])
        colour, z = (x + y + w) % 2, 6
    nB = N * dim
    Jb = (1 - 2 * _bits(_philox(np.arange(-(-nB // 128)), 0, 0, 5, spec["disorder_seed"]), nB)).reshape(N, dim)
    J = np.stack([Jb[:, a] for a in range(dim)] + [Jb[nb[dim + a], a] for a in range(dim)])
    R0 = R = spec["R0"]
    r = np.arange(R)
    s = 1 - 2 * _bits(_philox(np.arange(-(-N // 128))[None, :], r[:, None], 0, 1, seed), N)
    energy = lambda s: sum((Jb[:, a] * s * s[:, nb[a]]).sum(1) for a in range(dim))  # noqa: E731

    def sweeps(s, beta, t0):
        dEs = [4 * u - 2 * z for u in range(z + 1)]
        T = [1 << 64 if d <= 0 or math.exp(-beta * d) >= 1 else int(math.floor(math.ldexp(math.exp(-beta * d), 64))) for d in dEs]
        top, rep = np.array([t >> 48 for t in T], np.uint64), np.arange(len(s))
        for t in range(t0, t0 + c["n_sweeps"]):
            for col in range(2):
                site = i[colour == col]
                h = site // 2
                v = _philox(np.arange(-(-(N // 2) // 8))[None, :], rep[:, None], 2 * t + col, 2, seed)
                u = (v[..., None] >> np.array([0, 16], np.uint64)) & np.uint64(0xFFFF)
                u = u.reshape(len(s), -1)[:, h]
                cls = sum((J[a, site] * s[:, site] * s[:, nb[a][site]] < 0) for a in range(z)).astype(np.int64)
                acc = u < top[cls]
                for a, b in zip(*np.nonzero(u == top[cls])):
                    w = _philox(int(site[b]), int(a), 2 * t + col, 3, seed)
                    acc[a, b] = ((int(u[a, b]) << 48) | int(w[0]) | ((int(w[1]) & 0xFFFF) << 32)) < T[cls[a, b]]
                s[:, site] = np.where(acc, -s[:, site], s[:, site])
        return s

    betas = _betas(c)
    rec = np.zeros((c["n_steps"] + 1, 16))
    rec[0, 2], rec[0, 4] = N * math.log(2.0), R0
    if betas[0] > 0:
        s = sweeps(s, betas[0], c["n_steps"] * c["n_sweeps"])
    total = 0.0
    for k in range(1, len(betas)):
        E = energy(s)
        d = betas[k] - betas[k - 1]
        lo = int(E.min())
        wt = np.exp(-d * (E - lo))
        # equal terms are added as count times weight, energies ascending
        lev, cnt = np.unique(E, return_counts=True)
        wl = [math.exp(-d * float(e - lo)) for e in lev]
        S = 0.0
        for n, w in zip(cnt, wl):
            S += n * w
        wt = np.array(wl)[np.searchsorted(lev, E)]
        lnQ = -d * lo + math.log(S) - math.log(R)
        total += lnQ
        first = _philox(np.arange(2)[None, :], np.arange(R)[:, None], k, 4, seed).reshape(R, 8)
        cop = np.array([_copies(j, R0 * wt[j] / S, k, seed, first[j]) for j in range(R)])
        s = np.repeat(s, cop, axis=0)
        R = len(s)
        s = sweeps(s, betas[k], (k - 1) * c["n_sweeps"])
        E = energy(s).astype(np.float64)
        m = E.mean()
        m2, m3 = ((E - m) ** 2).mean(), ((E - m) ** 3).mean()
        rec[k, :9] = [betas[k], lnQ, N * math.log(2.0) + total, S, R, lo, m, m2, m3 / m2 ** 1.5 if m2 > 0 else 0.0]
    return rec
