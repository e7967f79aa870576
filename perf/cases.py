"""The work that users of this framework have it do, as cases to be timed.

A case is one call (or one run) through the Python binding of the C ABI, at
sizes from the smallest test run to the large single run: SMC runs (``run``),
many uneven runs advanced together (``batch``), posterior predictive bands
(``predict``), bare trajectories (``simulate``), the learned screen's network
forward on device buffers (``forward``) and its training (``train``).

``exact`` evaluates the method in 64 bits with plain torch operations (its own
Philox, samplers and sums, written from the method's definition), on the GPU
where there is one.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2106_15508_amd import abcsmc as A
from paper_2106_15508_amd import workloads as W

DEV = "cuda" if torch.cuda.is_available() else "cpu"


# ------------------------------------------------------------------- the cases

def run_case(population, days, particles, stages, *, early_exit=True, sampler="binomial", step="paper",
             surv=0.5, variance=False, **more):
    return dict(kind="run", population=population, days=days, particles=particles, stages=stages,
                early_exit=early_exit, sampler=sampler, step=step, surv=surv, variance=variance, **more)


def listed():
    return [
        # the smallest run of the tests: interactive use, all launch latency
        run_case(20_000, 30, 300, 4, early_exit=False, name="run tiny"),
        # the small published-size workload with fixed Beta(2, 5) step sizes
        run_case(100_000, 50, 1024, 4, step="fixed", name="run small fixed-beta"),
        # the paper's own transition sampler, step size read as a variance, a ragged particle count
        run_case(800_000, 75, 5003, 6, sampler="normal", variance=True, surv=0.4, name="run floor-normal ragged"),
        # an ordinary fit of one region's series on an odd particle count
        run_case(3_000_000, 97, 20_011, 8, name="run ordinary"),
        # the headline run of bench.py
        run_case(10_000_000, 120, 131_072, 10, name="run headline"),
        # the large single run's size (country-scale population, 180 days) over its first stages
        run_case(300_000_000, 180, 1_048_576, 3, name="run large"),
        # a handful of regions fitted together, small particle counts
        dict(kind="batch", runs=12, lg_lo=9, lg_hi=12, stages=6, name="batch small"),
        # the many-run workload: uneven populations, horizons and particle counts
        dict(kind="batch", runs=48, lg_lo=11, lg_hi=16, stages=6, name="batch uneven"),
        # predictive bands past the fitted horizon from a fitted population
        dict(kind="predict", population=10_000_000, days=120, particles=32_768, stages=3, horizon=150, quantiles=3,
             name="predict bands"),
        # forward trajectories of given parameter vectors (synthetic data, prior checks)
        dict(kind="simulate", population=10_000_000, days=120, vectors=4096, name="simulate prior draws"),
        # scoring a pool of proposals with the screen's network, device to device
        dict(kind="forward", rows=65_536, name="network forward"),
        # fitting the network: a few passes over a training set
        dict(kind="train", rows=131_072, batch=32_768, epochs=2, name="network training"),
    ]


def log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run"] * 6 + ["batch"] * 2 + ["predict", "simulate", "forward", "train"])
    population, days = log_uniform(rng, 2e4, 3e8), rng.randint(25, 180)
    if kind == "run":
        particles = log_uniform(rng, 250, 300_000)
        most = 10 if particles < 150_000 else 5
        return run_case(population, days, particles, rng.randint(3, most), early_exit=rng.random() < 0.75,
                        sampler=rng.choice(["binomial"] * 4 + ["normal"]), step=rng.choice(["paper"] * 3 + ["fixed"]),
                        surv=rng.choice([0.3, 0.5, 0.5, 0.7]), variance=rng.random() < 0.15)
    if kind == "batch":
        lo = rng.randint(8, 13)
        return dict(kind=kind, runs=log_uniform(rng, 3, 48), lg_lo=lo, lg_hi=lo + rng.randint(1, 3),
                    stages=rng.randint(3, 6))
    if kind == "predict":
        return dict(kind=kind, population=population, days=days, particles=log_uniform(rng, 500, 60_000),
                    stages=rng.randint(1, 3), horizon=days + rng.randint(0, 60), quantiles=rng.choice([1, 3, 5]))
    if kind == "simulate":
        return dict(kind=kind, population=population, days=days, vectors=log_uniform(rng, 1, 20_000))
    if kind == "forward":
        return dict(kind=kind, rows=log_uniform(rng, 1, 65_536))
    return dict(kind=kind, rows=log_uniform(rng, 3000, 200_000), batch=rng.choice([1000, 2048, 8192, 32_768]),
                epochs=rng.randint(1, 3))


# ------------------------------------------------------------------ preparation

def workload(case, seed):
    """The workload of a run or predict case; every seed observes another series."""
    step = dict(step_schedule=W.STEP_FIXED, beta_a=2.0, beta_b=5) if case.get("step") == "fixed" else {}
    sampler = W.SAMPLER_NORMAL_FLOOR if case.get("sampler") == "normal" else W.SAMPLER_BINOMIAL
    return W.Workload("case", population=case["population"], n_days=case["days"], n_particles=case["particles"],
                      n_rounds=case["stages"], surv_ratio=case.get("surv", 0.5), sampler=sampler,
                      step_is_variance=bool(case.get("variance", False)), seed=1 + seed, obs_seed=210615508 + seed,
                      **step)


def batch_workloads(case, seed):
    """Uneven runs: their sizes belong to the case, their series and draws to the seed."""
    rng = np.random.default_rng([4, case["runs"], case["lg_lo"], case["lg_hi"]])
    ws = []
    for r in range(case["runs"]):
        ws.append(W.Workload(f"run{r}", population=int(round(math.exp(rng.uniform(math.log(1e5), math.log(3e8))))),
                             n_days=int(rng.integers(40, 151)),
                             n_particles=1 << int(rng.integers(case["lg_lo"], case["lg_hi"] + 1)),
                             n_rounds=case["stages"], seed=1000 + 100 * seed + r, obs_seed=210615508 + 400 + 100 * seed + r))
    return ws


def prior_vectors(case, seed):
    lo, hi = np.array(W.BENCH_LO), np.array(W.BENCH_HI)
    return lo + np.random.default_rng([5, seed]).random((case["vectors"], 8)) * (hi - lo)


def network_inputs(case, seed):
    """Network parameters at the scale of the initialisation, inputs 2u - 1 of
    unit-cube points, targets log1p of root sums of squares spanning the
    magnitudes a horizon of counts gives."""
    rng = np.random.default_rng([6, seed])
    parts = []
    for fan_out, fan_in in ((256, 8), (256, 256), (256, 256), (3, 256)):
        parts += [rng.standard_normal(fan_out * fan_in) / math.sqrt(fan_in), np.zeros(fan_out)]
    x = 2.0 * rng.random((case["rows"], 8)) - 1.0
    y = np.log1p(np.exp(6.0 + 4.0 * x[:, :3] - 2.0 * x[:, 3:6] * x[:, 5:8] + 0.3 * rng.standard_normal((case["rows"], 3))))
    return [v.astype(np.float32) for v in (np.concatenate(parts), x, y)]


def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case)
    if kind in ("run", "predict"):
        w = workload(case, seed)
        flags = A.F_EARLY_EXIT if case.get("early_exit", True) else 0
        state["ctx"] = A.Context(w, A.observations(w), flags=flags)
        if kind == "predict":
            state["ctx"].run(case["stages"])
            state["levels"] = levels(case)
            state["seed"] = 77 + seed
    elif kind == "batch":
        ws = batch_workloads(case, seed)
        state["batch"] = A.Batch(ws, [A.observations(w) for w in ws], flags=A.F_EARLY_EXIT)
    elif kind == "simulate":
        state["w"] = W.Workload("case", population=case["population"], n_days=case["days"], n_particles=2, n_rounds=1)
        state["theta"], state["seed"] = prior_vectors(case, seed), 900 + seed
    else:
        state["params"], state["x"], state["y"] = network_inputs(case, seed)
        if kind == "forward":
            for k in ("params", "x"):
                state[k] = torch.from_numpy(state[k]).cuda()
            state["out"] = torch.empty((case["rows"], 3), dtype=torch.float32, device="cuda")
    return state


def levels(case):
    return {1: (0.5,), 3: (0.005, 0.5, 0.995), 5: (0.005, 0.25, 0.5, 0.75, 0.995)}[case["quantiles"]]


# -------------------------------------------------------------------- one pass

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "run":
        ctx = state["ctx"]
        ctx.reset()
        infos = ctx.run(case["stages"])
        theta, dist, weight = ctx.weights()
        return dict(theta=theta, dist=dist, weight=weight, eps=np.array([i["eps_next"] for i in infos]),
                    ess=infos[-1]["ess"], proposals=np.array([i["proposals"] for i in infos], dtype=np.int64))
    if kind == "batch":
        b = state["batch"]
        b.reset()
        infos = b.run(case["stages"])
        pops = [b.population(r) for r in range(b.R)]
        out = {k: np.concatenate([p[k] for p in pops]) for k in ("u", "d", "W", "logw", "index", "parent")}
        out["eps"] = np.array([[i["eps_next"] for i in stage] for stage in infos])
        return out
    if kind == "predict":
        return state["ctx"].predict(case["horizon"], state["seed"], state["levels"])
    if kind == "simulate":
        return A.simulate(state["w"], state["theta"], state["seed"], 3)
    if kind == "forward":
        A.mlp_forward_noalloc(state["params"].data_ptr(), case["rows"], state["x"].data_ptr(), state["out"].data_ptr(),
                              torch.cuda.current_stream().cuda_stream)
        return state["out"]
    params, losses = A.mlp_train(state["params"], state["x"], state["y"], case["batch"], case["epochs"], 1e-3)
    return dict(params=params, losses=losses)


# ------------------------------------------------------------------------ work

#: multiply-adds of the network per row, and its parameters
MACS, PARAMS = 8 * 256 + 2 * 256 * 256 + 256 * 3, 134_659
#: FP64 operations of one simulated day and of one term of an importance-weight sum
DAY, TERM = 450, 58


def work(case):
    """Bytes: inputs once and outputs once.  Operations: every accepted
    particle's simulation, and of the weight sums a tenth of the (particle,
    surviving parent) pairs (the others are below the sums' rounding)."""
    kind = case["kind"]
    if kind in ("run", "batch"):
        if kind == "run":
            sizes = [(case["particles"], case["days"])]
            surv = case["surv"]
        else:
            sizes, surv = [(w.n_particles, w.n_days) for w in batch_workloads(case, 0)], 0.5
        flops = sum(case["stages"] * n * t * DAY + (case["stages"] - 1) * 0.1 * n * n * surv * TERM for n, t in sizes)
        return dict(bytes=sum(80 * n + 24 * t for n, t in sizes), flops=flops)
    if kind == "predict":
        rows = 3 * (case["horizon"] + 1)
        return dict(bytes=64 * case["particles"] + 8 * rows * case["quantiles"],
                    flops=case["particles"] * case["horizon"] * DAY)
    if kind == "simulate":
        return dict(bytes=case["vectors"] * (64 + 48 * (case["days"] + 1)), flops=case["vectors"] * case["days"] * DAY)
    if kind == "forward":
        return dict(bytes=4 * (PARAMS + 11 * case["rows"]), flops=2 * MACS * case["rows"])
    return dict(bytes=4 * (2 * PARAMS + 11 * case["rows"]), flops=6 * MACS * case["rows"] * case["epochs"])


# ----------------------------------------------- the method in 64 bits, in torch

M32 = 0xFFFFFFFF
PRIOR, PERTURB, SIM = 1, 2, 3


def philox(seed, index, stage, purpose, step, block):
    """Two 64-bit words (as (low, high) 32-bit halves in int64) of Philox4x32-10
    at counter (index, stage, purpose << 24 | step, block), key = seed."""
    c0, c1 = index, torch.full_like(index, stage)
    c2, c3 = torch.full_like(index, (purpose << 24) | step), torch.full_like(index, 0) + block
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        m0, m1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2
        c0, c1, c2, c3 = ((m1 >> 32) & M32) ^ c1 ^ k0, m1 & M32, ((m0 >> 32) & M32) ^ c3 ^ k1, m0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return (c0, c1), (c2, c3)


def words(seed, index, stage, purpose, step, blocks):
    """Words 0 .. 2 blocks - 1 of each index's stream."""
    n = index.numel()
    blk = torch.arange(blocks, device=index.device).repeat_interleave(n)
    a, b = philox(seed, index.repeat(blocks), stage, purpose, step, blk)
    return [tuple(h[k * n:(k + 1) * n] for h in half) for k in range(blocks) for half in (a, b)]


def uniform(w):
    return (((w[1] << 20) | (w[0] >> 12)).double() + 0.5) * 2.0 ** -52


def normals(w):
    u1, u2 = (w[0].double() + 0.5) * 2.0 ** -32, (w[1].double() + 0.5) * 2.0 ** -32
    r = torch.sqrt(-2.0 * torch.log(u1))
    return r * torch.cos(2.0 * math.pi * u2), r * torch.sin(2.0 * math.pi * u2)


def binomial(n, p, w, z):
    flip = p > 0.5
    q = torch.where(flip, 1.0 - p, p)
    m = n * q
    x = torch.minimum(torch.floor((m + 0.5) + torch.sqrt(m * (1.0 - q)) * z).clamp(min=0.0), n)
    small = ((m < 10.0) & (n > 0) & (p > 0) & (p < 1)).nonzero()[:, 0]
    if small.numel():
        ns, qs, us = n[small], q[small], uniform((w[0][small], w[1][small]))
        f = torch.exp(ns * torch.log1p(-qs))
        total, r, k = f.clone(), qs / (1.0 - qs), torch.zeros_like(f)
        for it in range(128):
            on = (us > total) & (k < ns)
            if it % 8 == 0 and not bool(on.any()):
                break
            f = torch.where(on, f * (((ns - k) * r) * (1.0 / (it + 1))), f)
            k = k + on
            total = torch.where(on, total + f, total)
        x[small] = k
    x = torch.where(flip, n - x, x)
    x = torch.where(p >= 1.0, n, x)
    return torch.where((n <= 0) | (p <= 0), torch.zeros_like(x), x)


def floor_normal(n, h, w):
    x = torch.minimum(torch.floor(h + torch.sqrt(h.clamp(min=0.0)) * normals(w)[0]).clamp(min=0.0), n)
    return torch.where((n <= 0) | ~(h > 0), torch.zeros_like(x), x)


def trajectories(theta, population, days, sampler, seed, index, stage, start):
    """S, I, A, R, D, Ru of every vector, day after day."""
    a0, a1, ex, beta, gamma, delta, eta, kappa = theta.unbind(1)
    P = float(population)
    a, r, d = (torch.full_like(a0, float(v)) for v in start)
    i = torch.minimum(torch.floor(kappa * a), P - (a + r + d)).clamp(min=0.0)
    s, ru = P - (a + r + d + i), torch.zeros_like(a)
    rates = gamma, beta, delta, beta * eta
    probs = [-torch.expm1(-v) for v in rates]
    yield s, i, a, r, d, ru
    for t in range(days):
        c = a + r + d
        pw = torch.where(c == 0, (ex == 0).double(), torch.exp(ex * torch.log(c.clamp(min=1e-300))))
        rate = ((a0 + a1 / (1.0 + pw)) * i) * (1.0 / P)
        w = words(seed, index, stage, SIM, t, 4 if sampler == "binomial" else 3)
        if sampler == "binomial":
            (z0, z1), (z2, z3), (z4, _) = normals(w[5]), normals(w[6]), normals(w[7])
            n1, n2 = binomial(s, -torch.expm1(-rate), w[0], z0), binomial(i, probs[0], w[1], z1)
            n3 = binomial(a, probs[1], w[2], z2)
            n4, n5 = binomial(a - n3, probs[2], w[3], z3), binomial(i - n2, probs[3], w[4], z4)
        else:
            n1, n2 = floor_normal(s, rate * s, w[0]), floor_normal(i, rates[0] * i, w[1])
            n3 = floor_normal(a, rates[1] * a, w[2])
            n4, n5 = floor_normal(a - n3, rates[2] * a, w[3]), \
                floor_normal(i - n2, rates[3] * i, w[4])
        s, i, a, r, d, ru = s - n1, i + n1 - n2 - n5, a + n2 - n3 - n4, r + n3, d + n4, ru + n5
        yield s, i, a, r, d, ru


def box():
    lo, hi = (torch.tensor(v, dtype=torch.float64, device=DEV) for v in (W.BENCH_LO, W.BENCH_HI))
    return lo, hi - lo


def observed(w):
    """The synthetic series of the generating vector."""
    sampler = "normal" if w.sampler == W.SAMPLER_NORMAL_FLOOR else "binomial"
    theta = torch.tensor([w.theta_true], dtype=torch.float64, device=DEV)
    days = list(trajectories(theta, w.population, w.n_days, sampler, w.obs_seed,
                             torch.zeros(1, dtype=torch.int64, device=DEV), W.OBS_ROUND, w.obs0))
    return [torch.cat(x[2:5]) for x in days]


def distances(w, u, index, stage, obs):
    lo, width = box()
    sampler = "normal" if w.sampler == W.SAMPLER_NORMAL_FLOOR else "binomial"
    total = torch.zeros(len(u), dtype=torch.float64, device=DEV)
    for t, x in enumerate(trajectories(lo + u * width, w.population, w.n_days, sampler, w.seed, index, stage,
                                       [int(v) for v in obs[0]])):
        if t:
            for c in range(3):
                total += (x[2 + c] - obs[t][c]) ** 2
    return torch.sqrt(total)


def perturbed(w, stage, index, u_prev, cdf, shape_a, shape_b):
    """(u, sigma) of each index: the first in-cube attempt of at most 256."""
    n = index.numel()
    u = torch.zeros((n, 8), dtype=torch.float64, device=DEV)
    sigma, done = torch.zeros(n, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.bool, device=DEV)
    Q = int(cdf[-1])
    q0, q1 = Q & M32, Q >> 32
    left = torch.arange(n, device=DEV)
    for att in range(256):
        if not left.numel():
            break
        v = words(w.seed, index[left], stage, PERTURB, att, 3 + shape_b // 2)
        lo, hi = v[0]
        # high 64 bits of word * Q, from 32-bit halves; >> on the unsigned products
        p00, p01, p10 = lo * q0, lo * q1, hi * q0
        mid = ((p00 >> 32) & M32) + (p01 & M32) + (p10 & M32)
        r = hi * q1 + ((p01 >> 32) & M32) + ((p10 >> 32) & M32) + (mid >> 32)
        k = torch.searchsorted(cdf, r, right=True)
        L = torch.zeros(left.numel(), dtype=torch.float64, device=DEV)
        for m in range(shape_b):
            L += torch.log(uniform(v[5 + m])) / (shape_a + m)
        s = torch.exp(L)
        s = (torch.sqrt(s) if w.step_is_variance else s).clamp(min=1e-8)
        z = torch.stack([x for j in range(1, 5) for x in normals(v[j])], 1)
        new = u_prev[k] + s[:, None] * z
        ok = ((new >= 0) & (new <= 1)).all(1)
        u[left[ok]], sigma[left[ok]], done[left[ok]] = new[ok], s[ok], True
        left = left[~ok]
    return u, sigma, done


def smc(w, stages, want_weights=True):
    """The run in 64 bits: u, d, normalised weights, tolerances, effective
    sample size, proposals."""
    obs, N = observed(w), w.n_particles
    eps, eps1, eps_list, props = math.inf, math.inf, [], []
    for stage in range(stages):
        got, base, rate = [], 0, 0.8
        if stage:
            strict = bool((d < eps).any())
            wt = torch.where(d < eps if strict else d <= eps, eps - d, torch.full_like(d, -1.0))
            top = float(wt.max())
            q = torch.floor(wt / top * 2.0 ** 40).clamp(min=0).long() if top > 0 else (wt >= 0).long()
            cdf, u_prev = torch.cumsum(q, 0), u
            eps1 = eps if stage == 1 else eps1
            shape = (w.beta_a, w.beta_b) if w.step_schedule == W.STEP_FIXED else (eps / eps1, 2 * stage)
        have = 0
        while have < N:
            count = N - have if stage == 0 else int((N - have) / rate * 1.1) + 256
            index = torch.arange(base, base + count, device=DEV)
            if stage == 0:
                u = torch.stack([uniform(v) for v in words(w.seed, index, 0, PRIOR, 0, 4)], 1)
                sigma, ok = torch.zeros(count, dtype=torch.float64, device=DEV), torch.ones(count, dtype=torch.bool, device=DEV)
            else:
                u, sigma, ok = perturbed(w, stage, index, u_prev, cdf, *shape)
            d = distances(w, u, index, stage, obs)
            ok &= d <= eps
            got.append((u[ok], d[ok], sigma[ok], index[ok]))
            have += int(ok.sum())
            base += count
            rate = max(have / base, 1e-3)
        u, d, sigma, index = (torch.cat(x)[:N] for x in zip(*got))
        props.append(int(index[-1]) + 1)
        eps = float(np.quantile(d.cpu().numpy(), w.surv_ratio))
        eps_list.append(eps)
    W_, ess = torch.full((N,), 1.0 / N, dtype=torch.float64, device=DEV), float(N)
    if want_weights and stages > 1:
        keep = q > 0
        cols, logq = u_prev[keep], torch.log(q[keep].double())
        logw = torch.empty(N, dtype=torch.float64, device=DEV)
        step = max(1, (1 << 26) // len(cols))
        for b in range(0, N, step):
            d2 = torch.zeros((min(step, N - b), len(cols)), dtype=torch.float64, device=DEV)
            for c in range(8):
                d2.add_((u[b:b + step, c:c + 1] - cols[None, :, c]).square_())
            d2.mul_(-0.5 / sigma[b:b + step, None] ** 2).add_(logq)
            logw[b:b + step] = 8.0 * torch.log(sigma[b:b + step]) - torch.logsumexp(d2, 1)
        W_ = torch.softmax(logw, 0)
        ess = float(1.0 / (W_ * W_).sum())
    return u, d, W_, np.array(eps_list), ess, np.array(props, dtype=np.int64)


def network(params, x):
    """The network in 64 bits on torch parameters: the layers' weights and biases."""
    at, shapes = 0, ((256, 8), (256, 256), (256, 256), (3, 256))
    h = x
    for layer, (o, i) in enumerate(shapes):
        Wt, b = params[at:at + o * i].view(o, i), params[at + o * i:at + o * i + o]
        at += o * i + o
        h = torch.nn.functional.linear(h, Wt, b)
        if layer < 3:
            h = torch.nn.functional.gelu(h, approximate="tanh")
    return h


def exact(case, seed):
    kind = case["kind"]
    if kind in ("run", "predict"):
        steps = case["stages"] * case["days"] + (case["horizon"] if kind == "predict" else 0)
        # about 10 us an operation, about 1000 a simulated day; larger arrays cost their traffic
        if steps * (1.0 + case["particles"] / 1e5) > 3000 or case["particles"] > 200_000:
            return None
        w = workload(case, seed)
        u, d, weight, eps, ess, props = smc(w, case["stages"], want_weights=kind == "run")
        lo, width = box()
        if kind == "run":
            return dict(theta=lo + u * width, dist=d, weight=weight, eps=eps, ess=ess, proposals=props)
        start = [w.a0, 0, 0]
        index = torch.arange(len(u), device=DEV)
        series = trajectories(lo + u * width, w.population, case["horizon"], "binomial", 77 + seed, index, 0xFFFE, start)
        q = np.array(levels(case))
        return np.stack([np.quantile(torch.stack(x[2:5]).cpu().numpy(), q, axis=1).T for x in series])
    if kind == "simulate":
        theta = torch.from_numpy(prior_vectors(case, seed)).to(DEV)
        a0 = max(10, int(math.floor(1e-5 * case["population"])))
        days = trajectories(theta, case["population"], case["days"], "binomial", 900 + seed,
                            torch.arange(len(theta), device=DEV), 3, (a0, 0, 0))
        return torch.stack([torch.stack(x, 1) for x in days], 1).long()
    if kind == "batch":
        return None  # one run after another in torch takes minutes
    params, x, y = (torch.from_numpy(v).to(DEV).double() for v in network_inputs(case, seed))
    if kind == "forward":
        return network(params, x)
    params.requires_grad_(True)
    opt = torch.optim.Adam([params], lr=1e-3, betas=(0.9, 0.999), eps=1e-8)
    losses = []
    for _ in range(case["epochs"]):
        total = 0.0
        for b in range(0, case["rows"], case["batch"]):
            xb, yb = x[b:b + case["batch"]], y[b:b + case["batch"]]
            loss = torch.nn.functional.mse_loss(network(params, xb), yb)
            opt.zero_grad()
            loss.backward()
            opt.step()
            total += float(loss.detach()) * len(xb)
        losses.append(total / case["rows"])
    return dict(params=params.detach(), losses=np.array(losses))
