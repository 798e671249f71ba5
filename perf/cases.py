"""Cases that measure the library: what a user's program has it do, through the public entry points.

Every case is one of six uses, named by its "kind":

  run       es.run(T): many generations in one call, the loop of a benchmark or a hyper-parameter sweep
  step      es.ask(), es.eval(), es.tell(): one generation with a built-in problem, the loop of a program that
            looks at each generation's fitness
  external  es.ask(materialize=True), es.tell(fitness): the population handed out and a fitness that the program
            computed itself (a simulator) handed back
  tell      es.ask(), es.tell(fitness): the same where the program makes the population by itself; ranks and
            weights are read back with es.shaped()
  noalloc   eval_noalloc(): the evaluate without a handle, for callers that cannot allocate
  mlp       one generation of the neuroevolution problem (64-256-256-16 network against a teacher)

The state (mean, moments, generation) is drawn from the seed as a search some way in has it: the mean within the
problem's range, first and second moments at the size that the gradient estimate has there.  The listed sizes are
the workloads of paper_2212_04180_amd.workloads and generic ragged ones; draw() spreads over the ranges between.

exact() repeats the arithmetic (the Philox-4x32-10 stream of key seed + run and counter (d / 4, row, t, domain),
Box-Muller, the problems, shaping, gradient and update rules of include/esmi.h) in 64 bits.  What follows from
ranks of the library's own fitness (the state after a generation of kind run, step or mlp) has no such value: two
members whose fitnesses lie within the fitness's rounding may take either order, and the gradient follows it.
"""
from __future__ import annotations

import math

import torch

import paper_2212_04180_amd as P

PROBLEMS = {"none": P.PROB_NONE, "sphere": P.PROB_SPHERE, "shifted_sphere": P.PROB_SHIFTED_SPHERE,
            "rosenbrock": P.PROB_ROSENBROCK, "rastrigin": P.PROB_RASTRIGIN, "mlp": P.PROB_MLP}
STRATEGIES = {"openai": P.STRAT_OPENAI_ES, "pgpe": P.STRAT_PGPE, "snes": P.STRAT_SNES, "sepcma": P.STRAT_SEP_CMA}
SHAPINGS = {"ranks": P.SHAPE_CENTERED_RANK, "raw": P.SHAPE_RAW, "zscore": P.SHAPE_Z_SCORE}
RANGE = {"none": 3.0, "sphere": 5.0, "shifted_sphere": 2.0, "rosenbrock": 2.0, "rastrigin": 5.12}  # |mean| at the start
T0 = 50  # generations behind the drawn state
MLP_LAYERS = (64, 256, 256, 16)
MLP_PARAMS = 86544
MLP_BATCH = 256


def _case(kind, problem, D, N, R=1, T=1, sigma=0.1, lr=0.01, strategy="openai", optimizer="adam", shaping="ranks",
          w_decay=0.0, name=None):
    c = {"kind": kind, "problem": problem, "D": D, "N": N, "R": R, "T": T, "sigma": sigma, "lr": lr,
         "strategy": strategy, "optimizer": optimizer, "shaping": shaping, "w_decay": w_decay}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest: one low-dimensional benchmark run, all latency
        _case("run", "sphere", 16, 32, T=100, name="run_sphere_d16"),
        # one run too large for a workgroup and far too small for the chip
        _case("run", "rosenbrock", 1000, 256, T=500, sigma=0.05, lr=0.005, name="run_rosenbrock_d1000"),
        # a sweep over seeds: a thousand small runs at once
        _case("run", "rastrigin", 100, 64, R=1024, T=200, sigma=0.2, lr=0.02, name="run_rastrigin_r1024"),
        # the same medium problem a generation at a time: launches count
        _case("step", "rosenbrock", 1000, 256, sigma=0.05, lr=0.005, name="step_rosenbrock_d1000"),
        # the headline: one very large search
        _case("step", "shifted_sphere", 1_000_000, 2048, sigma=0.01, lr=0.001, name="step_sphere_d1m"),
        # the other strategies, ragged sizes, per-dimension sigma or independent members
        _case("step", "shifted_sphere", 250_003, 1000, sigma=0.01, lr=0.05, strategy="pgpe", optimizer="clipup",
              name="step_pgpe_d250003"),
        _case("step", "rastrigin", 100_001, 510, R=2, sigma=0.05, lr=1.0, strategy="snes", name="step_snes_d100001"),
        _case("step", "sphere", 50_001, 510, sigma=0.05, strategy="sepcma", name="step_sepcma_d50001"),
        # a simulator's fitness: the population is written out
        _case("external", "none", 10_007, 1024, R=2, sigma=0.05, shaping="zscore", w_decay=0.005,
              name="external_d10007"),
        # a very large population of a small network
        _case("tell", "none", 50, 65_536, sigma=0.05, name="tell_n65536"),
        # several searches evaluated inside somebody else's serving loop
        _case("noalloc", "rastrigin", 20_000, 1000, R=4, sigma=0.1, name="noalloc_rastrigin_r4"),
        # neuroevolution: matrix work per member
        _case("mlp", "mlp", MLP_PARAMS, 1024, sigma=0.02, name="mlp_n1024"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _even(x):
    return max(2, 2 * int(x / 2))


def draw(rng):
    kind = rng.choice(("run", "run", "run", "step", "step", "step", "external", "tell", "noalloc", "mlp"))
    if kind == "mlp":
        return _case("mlp", "mlp", MLP_PARAMS, _even(_log(rng, 64, 1024)), sigma=rng.choice((0.02, 0.05)),
                     strategy=rng.choice(("openai", "openai", "pgpe")), optimizer=rng.choice(("adam", "clipup")))
    problem = rng.choice(("sphere", "shifted_sphere", "rosenbrock", "rastrigin"))
    sigma = rng.choice((0.02, 0.05, 0.1, 0.2))
    lr = rng.choice((0.005, 0.01, 0.02))
    if kind == "run":
        while True:
            D, N, R = int(_log(rng, 4, 4000)), _even(_log(rng, 16, 1024)), int(_log(rng, 1, 1024))
            T = int(rng.uniform(20, 200))
            work = D * N * R  # member-dims of a generation: as much as the listed runs
            if work <= 6_600_000 and work * T <= 6_600_000 * 60:
                return _case("run", problem, D, N, R=R, T=T, sigma=sigma, lr=lr)
    if kind == "step":
        strategy = rng.choice(("openai", "openai", "openai", "pgpe", "snes", "sepcma"))
        optimizer = rng.choice(("adam", "adam", "clipup")) if strategy in ("openai", "pgpe") else "adam"
        while True:
            D, N, R = int(_log(rng, 200, 1_000_000)), _even(_log(rng, 32, 2048)), int(_log(rng, 1, 8))
            if 200_000 <= D * N * R <= 700_000_000:
                break
        shaping, w_decay = ("ranks", 0.0) if strategy != "openai" else rng.choice((("ranks", 0.0), ("ranks", 0.005),
                                                                                   ("zscore", 0.0)))
        return _case("step", problem, D, N, R=R, sigma=sigma, lr=1.0 if strategy == "snes" else lr, strategy=strategy,
                     optimizer=optimizer, shaping=shaping, w_decay=w_decay)
    if kind == "external":
        while True:
            D, N, R = int(_log(rng, 100, 200_000)), _even(_log(rng, 32, 2048)), int(_log(rng, 1, 4))
            if 100_000 <= D * N * R <= 60_000_000:
                break
        return _case("external", "none", D, N, R=R, sigma=sigma, lr=lr, strategy=rng.choice(("openai", "pgpe")),
                     optimizer=rng.choice(("adam", "clipup")), shaping=rng.choice(("ranks", "zscore")))
    if kind == "tell":
        return _case("tell", "none", int(_log(rng, 10, 500)), _even(_log(rng, 4000, 100_000)), sigma=sigma, lr=lr,
                     strategy=rng.choice(("openai", "snes", "pgpe")))
    while True:
        D, N, R = 4 * int(_log(rng, 100, 50_000)), _even(_log(rng, 32, 2048)), int(_log(rng, 1, 8))
        if 200_000 <= D * N * R <= 400_000_000:
            return _case("noalloc", problem, D, N, R=R, sigma=sigma)


# ---- inputs ---------------------------------------------------------------------------------------------------
def _config(case, seed):
    c = case
    init = P.INIT_FANIN_NORMAL if c["kind"] == "mlp" else P.INIT_ZERO
    snes_lr = (3.0 + math.log(c["D"])) / (5.0 * math.sqrt(c["D"]))
    return P.ESConfig(num_dims=c["D"], popsize=c["N"], num_runs=c["R"], sigma=c["sigma"], lr=c["lr"],
                      seed=1000 + 7919 * (seed % 1_000_003), init=init, problem=PROBLEMS[c["problem"]],
                      maximize=1 if c["kind"] == "mlp" else 0, strategy=STRATEGIES[c["strategy"]],
                      optimizer=P.OPT_CLIPUP if c["optimizer"] == "clipup" else P.OPT_ADAM,
                      shaping=SHAPINGS[c["shaping"]], w_decay=c["w_decay"],
                      sigma_lr=snes_lr if c["strategy"] == "snes" else 0.2, clipup_max_speed=0.3)


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _inputs(case, seed):
    """Mean, moments, per-dimension sigma, velocity [R][D] and fitness [R][N], fp32 on the device, from the seed."""
    dev = _device()
    gen = torch.Generator(dev).manual_seed(int(seed))
    R, D, N = case["R"], case["D"], case["N"]

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float32)

    def uniform(*shape):
        return torch.rand(*shape, generator=gen, device=dev, dtype=torch.float32)

    if case["kind"] == "mlp":
        m = normal(R, D) * _mlp_scale(dev).float()
    else:
        m = (2.0 * uniform(R, D) - 1.0) * RANGE[case["problem"]]
    # the gradient estimate's size under centered ranks: sqrt(N / 12) / (N sigma) per dimension
    g = 0.29 / (case["sigma"] * math.sqrt(N))
    if case["strategy"] == "sepcma":
        m1, v = normal(R, D), 0.3 * normal(R, D)  # the evolution paths
    else:
        m1, v = 0.5 * g * normal(R, D), g * g * (0.5 + uniform(R, D))
    sig = case["sigma"] * (0.7 + 0.6 * uniform(R, D))
    if case["strategy"] == "sepcma":
        sig = 0.7 + 0.6 * uniform(R, D)  # the diagonal covariance
    vel = 0.1 * normal(R, D) / math.sqrt(D)
    fit = 10.0 + 3.0 * normal(R, N)
    fit = torch.where(uniform(R, N) < 0.05, torch.round(fit), fit)  # some members tie
    return {"m": m, "m1": m1, "v": v, "sig": sig, "vel": vel, "fit": fit}


def prepare(case, seed):
    cfg, x = _config(case, seed), _inputs(case, seed)
    if case["kind"] == "noalloc":
        shift = None
        if case["problem"] == "shifted_sphere":
            shift = P.ES(_config(case, seed)).problem_data()
        sigma = torch.full((case["R"],), case["sigma"], device=x["m"].device)
        return {"kind": "noalloc", "cfg": cfg, "m": x["m"], "sigma": sigma, "shift": shift, "t": T0}
    es = P.ES(cfg)
    es.set_state(x["m"], x["m1"], x["v"], T0)
    vec = case["strategy"] != "openai"
    clip = case["optimizer"] == "clipup" and case["strategy"] in ("openai", "pgpe")
    if vec or clip:
        es.set_strategy_state(x["sig"] if vec else None, x["vel"] if clip else None)
    return {"kind": case["kind"], "es": es, "T": case["T"], "fit": x["fit"], "vec": vec, "clip": clip}


def run(state):
    kind = state["kind"]
    if kind == "noalloc":
        return P.eval_noalloc(state["cfg"], state["m"], state["sigma"], state["t"], state["shift"])
    es, out = state["es"], {}
    if kind == "run":
        out["log"] = es.run(state["T"])
    elif kind in ("step", "mlp"):
        es.ask()
        out["fitness"] = es.eval()
        es.tell(out["fitness"])
    else:
        out["x"] = es.ask(materialize=kind == "external")
        es.tell(state["fit"])
        if kind == "tell":
            out["y"], out["rank"] = es.shaped()
    st = es.get_state()
    out["m"], out["m1"], out["v"] = st["m"], st["m1"], st["v"]
    if state["vec"] or state["clip"]:
        out["sigma"], out["velocity"] = es.strategy_state(sigma=state["vec"], velocity=state["clip"])
    return out


# ---- what a pass cannot do without ---------------------------------------------------------------------------
def work(case):
    R, D, N, kind = case["R"], case["D"], case["N"], case["kind"]
    gens = case["T"] if kind == "run" else 1
    rows = N if case["strategy"] == "sepcma" else N // 2
    normals = float(R) * rows * D
    members = float(R) * N * D
    # per normal: a quarter of a Philox block (20 products, 40 xors) and of two Box-Muller pairs (26 operations)
    flops = normals * 21.5
    terms = {"none": 0, "mlp": 0, "sphere": 4, "shifted_sphere": 5, "rosenbrock": 9, "rastrigin": 8}[case["problem"]]
    flops += members * terms
    if kind != "noalloc":
        flops += normals * (2 if case["strategy"] == "openai" else 6)  # the weighted sums over the population
    if kind == "mlp":
        flops += float(R) * N * 2 * MLP_BATCH * (64 * 256 + 256 * 256 + 256 * 16)
    state = 4.0 * R * D
    nbytes = 4.0 * R * N + state  # the fitness, the mean
    if kind != "noalloc":
        nbytes += 5 * state  # the moments read, the state written
    if case["strategy"] != "openai":
        nbytes += 2 * state
    if case["problem"] in ("shifted_sphere", "mlp"):
        nbytes += 4.0 * D
    if kind == "external":
        nbytes += 4.0 * members
    if kind == "run":
        nbytes += 4.0 * R * gens
    if kind == "tell":
        nbytes += 12.0 * R * N
    return {"bytes": nbytes, "flops": flops * gens}


def tolerance(case):
    """Four times what the sums in another order (shorter evaluate chunks, another split of the gradient) change.

    One evaluate or one update: 32-bit sums, 1e-7 measured against 64 bits.  A generation whose ranks come from the
    library's own fitness: two members within the fitness's rounding change places, which moved the first moments
    and the velocity by 2e-4 to 6e-4.  A whole run collects such changes: 7e-3 in the first moments of a thousand
    64-member runs after 200 generations (their mean by 4e-5, a single value by 0.19), 3e-3 with 18 members.
    """
    kind = case["kind"]
    if kind == "run":
        return {"rel": 2.7e-2, "max": 0.75}
    if kind in ("step", "mlp"):
        return {"rel": 5e-3, "max": 5e-2}
    return {"rel": 2e-6, "max": 2e-5}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _philox(key, c0, c1, c2, c3):
    """Philox-4x32-10 words (int64 tensors holding 32-bit values)."""
    k0, k1 = key & _M32, (key >> 32) & _M32

    def product(c, mul):  # low and high word of the 64-bit product (int64 arithmetic wraps mod 2^64)
        p = c * (mul - (1 << 64) if mul >> 63 else mul)
        return p & _M32, (p >> 32) & _M32

    for _ in range(10):
        l0, h0 = product(c0, 0xD2511F53)
        l1, h1 = product(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1, c2, c3


def _normals(key, rows, nblocks, t, domain, dev):
    """[rows][4 nblocks] fp64 standard normals."""
    c0 = torch.arange(nblocks, device=dev, dtype=torch.int64)[None, :].expand(len(rows), nblocks)
    c1 = rows[:, None].expand(len(rows), nblocks)
    w = _philox(key, c0, c1, torch.full_like(c0, t), torch.full_like(c0, domain))
    e = torch.empty(len(rows), nblocks, 4, dtype=torch.float64, device=dev)
    for k in (0, 2):
        r = torch.sqrt(-2.0 * torch.log(((w[k] >> 8) + 1).double() * 2.0 ** -24))
        th = (w[k + 1] >> 8).double() * (2.0 ** -24 * 2.0 * math.pi)
        e[:, :, k], e[:, :, k + 1] = r * torch.cos(th), r * torch.sin(th)
    return e.reshape(len(rows), 4 * nblocks)


def _terms(problem, x, shift, a=10.0):
    if problem == "sphere":
        return (x * x).sum(-1)
    if problem == "shifted_sphere":
        return ((x - shift) ** 2).sum(-1)
    if problem == "rosenbrock":
        return (100.0 * (x[..., 1:] - x[..., :-1] ** 2) ** 2 + (1.0 - x[..., :-1]) ** 2).sum(-1)
    return (a + x * x - a * torch.cos(2.0 * math.pi * x)).sum(-1)


def _mlp_scale(dev):
    s = torch.zeros(MLP_PARAMS, dtype=torch.float64, device=dev)
    at = 0
    for i, o in zip(MLP_LAYERS[:-1], MLP_LAYERS[1:]):
        s[at:at + i * o] = 1.0 / math.sqrt(i)
        at += i * o + o
    return s


def _mlp(w, x):
    """Outputs [B][256][16] of networks w [B][86544] on the inputs x [256][64]."""
    h, at = x.expand(len(w), *x.shape), 0
    for k, (i, o) in enumerate(zip(MLP_LAYERS[:-1], MLP_LAYERS[1:])):
        wt = w[:, at:at + i * o].reshape(-1, o, i).transpose(1, 2).contiguous()
        at += i * o
        h = torch.bmm(h.contiguous(), wt) + w[:, None, at:at + o]
        at += o
        if k < 2:
            h = torch.tanh(h)
    return h


def _exact_parts(case, seed, weights=None):
    """Per run: fitness [N] (weights None), or the noise sums of the folded weights (a, b) of each run."""
    cfg, x, dev = _config(case, seed), _inputs(case, seed), _device()
    D, N, R = case["D"], case["N"], case["R"]
    nb, half = (D + 3) // 4, N // 2
    step = max(1, min(half, (1 << 22) // nb)) if case["kind"] != "mlp" else 16
    base = cfg.seed
    shift = teacher = inputs = None
    if case["problem"] == "shifted_sphere":
        shift = _normals(base, torch.zeros(1, dtype=torch.int64, device=dev), nb, 0, 2, dev)[0, :D]
    if case["kind"] == "mlp":
        flat = _normals(base, torch.zeros(1, dtype=torch.int64, device=dev), nb, 0, 2, dev)[0, :D] * _mlp_scale(dev)
        inputs = _normals(base, torch.zeros(1, dtype=torch.int64, device=dev), MLP_BATCH * 16, T0, 3, dev)
        inputs = inputs.reshape(MLP_BATCH, 64)
        teacher = _mlp(flat[None], inputs)
    got = []
    for r in range(R):
        m = x["m"][r].double()
        if case["strategy"] == "openai":
            s = torch.full_like(m, float(torch.tensor(case["sigma"], dtype=torch.float32)))
        elif case["strategy"] == "sepcma":
            s = float(torch.tensor(case["sigma"], dtype=torch.float32)) * torch.sqrt(x["sig"][r].double())
        else:
            s = x["sig"][r].double()
        fit = torch.empty(N, dtype=torch.float64, device=dev)
        A, B = torch.zeros_like(m), torch.zeros_like(m)
        for p in range(0, half, step):
            rows = torch.arange(p, min(half, p + step), device=dev, dtype=torch.int64)
            e = _normals(base + r, rows, nb, T0, 0, dev)[:, :D]
            if weights is not None:
                a, b = weights[r]
                A += (a[rows][:, None] * e).sum(0)
                B += (b[rows][:, None] * (e * e - 1.0)).sum(0)
                continue
            e2 = -e if case["strategy"] != "sepcma" else _normals(base + r, rows + half, nb, T0, 0, dev)[:, :D]
            for z, off in ((e, 0), (e2, half)):
                if case["kind"] == "mlp":
                    f = -((_mlp(m + s * z, inputs) - teacher) ** 2).mean((1, 2))
                else:
                    f = _terms(case["problem"], m + s * z, shift)
                fit[rows + off] = f
        got.append(fit if weights is None else (A, B))
    return got


def _exact_ask(case, seed):
    cfg, x, dev = _config(case, seed), _inputs(case, seed), _device()
    half, nb = case["N"] // 2, (case["D"] + 3) // 4
    out = torch.empty(case["R"], case["N"], case["D"], dtype=torch.float64, device=dev)
    for r in range(case["R"]):
        s = x["sig"][r].double() if case["strategy"] != "openai" else float(
            torch.tensor(case["sigma"], dtype=torch.float32))
        for p in range(0, half, 256):
            rows = torch.arange(p, min(half, p + 256), device=dev, dtype=torch.int64)
            e = s * _normals(cfg.seed + r, rows, nb, T0, 0, dev)[:, :case["D"]]
            out[r, rows] = x["m"][r].double() + e
            out[r, rows + half] = x["m"][r].double() - e
    return out


def _exact_tell(case, seed, pop=None):
    """The tell of kinds external and tell, from the given fitness."""
    cfg, x, dev = _config(case, seed), _inputs(case, seed), _device()
    R, N = case["R"], case["N"]
    half = N // 2
    f32 = lambda v: float(torch.tensor(v, dtype=torch.float32))  # noqa: E731
    key = x["fit"].double()
    if case["w_decay"]:
        key = key + f32(case["w_decay"]) * (pop * pop).mean(-1)
    rank = torch.argsort(torch.argsort(key, dim=1, stable=True), dim=1)
    if case["strategy"] == "snes":
        u = torch.exp(cfg.snes_temperature * ((N - 1 - rank).double() / N - 0.5))
        y = u / u.sum(1, keepdim=True)
    elif case["shaping"] == "zscore":
        y = (key - key.mean(1, keepdim=True)) / (key.std(1, unbiased=False, keepdim=True) + 1e-10)
    else:
        y = (2.0 * rank.double() - (N - 1)) / (2.0 * (N - 1))
    a, b = y[:, :half] - y[:, half:], y[:, :half] + y[:, half:]
    if case["strategy"] == "pgpe":
        b = b / 2.0 - y.mean(1, keepdim=True)
    sums = _exact_parts(case, seed, [(a[r], b[r]) for r in range(R)])
    A, B = torch.stack([s[0] for s in sums]), torch.stack([s[1] for s in sums])
    m, m1, v, sig, vel = (x[k].double() for k in ("m", "m1", "v", "sig", "vel"))
    lr, out = f32(case["lr"]), {"y": y, "rank": rank}
    if case["strategy"] == "snes":
        out.update(m=m + lr * sig * A, m1=m1, v=v, sigma=sig * torch.exp(0.5 * f32(cfg.sigma_lr) * B))
        return out
    g = sig * A / N if case["strategy"] == "pgpe" else A / (N * f32(case["sigma"]))
    if case["strategy"] == "pgpe":
        d = -f32(cfg.sigma_lr) * sig * B / half
        lim = f32(cfg.sigma_max_change) * sig
        out["sigma"] = sig + torch.minimum(torch.maximum(d, -lim), lim)
    if case["optimizer"] == "clipup":
        vel = lr * g / g.norm(dim=1, keepdim=True) + f32(cfg.clipup_momentum) * vel
        n = vel.norm(dim=1, keepdim=True)
        vel = torch.where(n > f32(cfg.clipup_max_speed), vel * f32(cfg.clipup_max_speed) / n, vel)
        out.update(m=m - vel, m1=m1, v=v, velocity=vel)
        return out
    b1, b2 = f32(cfg.beta1), f32(cfg.beta2)
    m1, v = b1 * m1 + (1 - b1) * g, b2 * v + (1 - b2) * g * g
    step = (m1 / (1 - b1 ** (T0 + 1))) / (torch.sqrt(v / (1 - b2 ** (T0 + 1))) + f32(cfg.eps))
    out.update(m=m - lr * step, m1=m1, v=v)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "run":
        return None  # many generations, each on the ranks of its own rounded fitness
    if kind == "noalloc":
        return torch.stack(_exact_parts(case, seed))
    if kind in ("step", "mlp"):
        out = {"fitness": torch.stack(_exact_parts(case, seed)), "m": None, "m1": None, "v": None}
        if case["strategy"] != "openai" or case["optimizer"] == "clipup":
            out.update(sigma=None, velocity=None)
        return out
    x = _exact_ask(case, seed) if kind == "external" else None
    got = _exact_tell(case, seed, x)
    out = {"x": x, "m": got["m"], "m1": got["m1"], "v": got["v"]}
    if kind == "tell":
        out["y"], out["rank"] = got["y"], got["rank"]
    if case["strategy"] != "openai" or case["optimizer"] == "clipup":
        out.update(sigma=got.get("sigma"), velocity=got.get("velocity"))
    return out
