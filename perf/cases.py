"""Solves that stand for what a program has this library do, with their sizes.

listed() names them, draw() gives more of the same ranges, prepare() makes
what a program holds before the call (the problem, and for the device entry
points its buffers), run() is one solve through a public entry point, work()
the arithmetic and traffic a solve cannot do without, and exact() the swarm
phase in plain numpy for the solves that return it.

A case is a dict:
  entry      "host"    zeus_minimize into host arrays
             "device"  zeus_minimize_async into device buffers
             "plan"    a captured plan (zeus_plan_*), replayed
             "batch"   zeus_minimize_batch of a stream of uneven requests
             "served"  a zeus_server given a stream of requests at once
             "user"    zeus_minimize_user of a compiled user objective
  objective, dim, n, lower, upper, iter_pso, iter_bfgs, ...  problem fields
  swarm      the swarm state is returned as well
  requests, stream, n_div   batch and served: the stream's length and number
             (which sizes it has), and what its start counts are divided by
  source     user: "rosenbrock" or "poisson"
"""
import numpy as np
import torch

from paper_2603_28770_amd import user_objectives as U
from paper_2603_28770_amd import workloads as W
from paper_2603_28770_amd import zeus as Z

_BOX = dict(W.BOXES, goldstein_price=(-2.0, 2.0))


def _case(name, entry, objective, dim, n, iter_pso, iter_bfgs, **kw):
    lo, hi = _BOX.get(objective, (-5.0, 5.0))
    c = {"entry": entry, "objective": objective, "dim": dim, "n": n, "lower": lo, "upper": hi,
         "iter_pso": iter_pso, "iter_bfgs": iter_bfgs}
    if name:
        c = {"name": name, **c}
    c.update(kw)
    return c


def listed():
    return [
        # a single small fit, called from a program that waits for the answer:
        # the two-dimensional problem with 1,024 starts
        _case("rosenbrock_d2_n1024", "host", "rosenbrock", 2, 1024, 10, 100, w=0.7, c1=1.5, c2=1.5,
              v_half=1.0, armijo_c=1e-4, swarm=True),
        # the five-dimensional problem stopped at its 100th convergence
        _case("rastrigin_d5_n1024_c100", "host", "rastrigin", 5, 1024, 5, 1000,
              required_converged=100),
        # multimodal search with many starts in ten dimensions
        _case("rastrigin_d10_n65536", "device", "rastrigin", 10, 65536, 20, 1000),
        # the two fifty-dimensional problems (131,072 starts): few iterations
        # with transcendental terms, and many with cheap terms
        _case("ackley_d50_n131072", "device", "ackley", 50, 131072, 5, 2000),
        _case("rosenbrock_d50_n131072", "device", "rosenbrock", 50, 131072, 5, 2000),
        # dimensions whose inverse Hessian spans several wavefronts, and the
        # largest dimension the library takes
        _case("rosenbrock_d128_n16384", "device", "rosenbrock", 128, 16384, 2, 1000),
        _case("rosenbrock_d200_n8192", "device", "rosenbrock", 200, 8192, 2, 2000),
        _case("rosenbrock_d256_n509", "device", "rosenbrock", 256, 509, 2, 2000),
        # limited-memory runs of a large problem
        _case("rosenbrock_d200_n8192_m8", "device", "rosenbrock", 200, 8192, 2, 2000, lbfgs_m=8),
        # a job list of mixed objectives, d from 2 to 128 and 256 to 16,384
        # starts, solved in one call
        {"name": "uneven_batch_64", "entry": "batch", "requests": 64, "stream": 3, "n_div": 1},
        # a request stream in mixed precision through the server, d from 2 to
        # 200 and 64 to 4,096 starts
        {"name": "served_mix_24", "entry": "served", "requests": 24, "stream": 4, "n_div": 16},
        # a user's likelihood fit: run-time compiled code, four parameters
        _case("user_poisson_n65536", "user", "user", 4, 65536, 10, 1000, lower=0.0, upper=10.0,
              source="poisson"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


# most starts drawn for a dimension (the listed sizes bound them)
def _n_max(d, lbfgs):
    if lbfgs:
        return 65536 if d <= 64 else 8192
    return 65536 if d <= 64 else 12288 if d <= 128 else 6144 if d <= 200 else 400


def draw(rng):
    kind = rng.random()
    if kind < 0.08:
        return {"entry": "batch", "requests": rng.randint(5, 50), "stream": rng.randint(1, 99),
                "n_div": rng.choice((1, 2, 4))}
    if kind < 0.14:
        return {"entry": "served", "requests": rng.randint(5, 23), "stream": rng.randint(1, 99),
                "n_div": rng.choice((16, 32, 64))}
    if kind < 0.20:
        source = rng.choice(("rosenbrock", "poisson"))
        if source == "poisson":
            return _case(None, "user", "user", 4, _log_uniform(rng, 1000, 60000), rng.randint(0, 10),
                         1000, lower=0.0, upper=10.0, source=source)
        return _case(None, "user", "user", _log_uniform(rng, 2, 50), _log_uniform(rng, 1000, 16384),
                     rng.randint(0, 10), 1000, source=source)
    objective = rng.choice(W.MIX)
    entry = rng.choice(("device", "device", "device", "plan", "host"))
    d = _log_uniform(rng, 2, 256)
    if kind < 0.27:  # stopped at a number of convergences
        d = min(d, 10)
        n = _log_uniform(rng, 1024, 65536)
        return _case(None, entry, objective, d, n, rng.randint(0, 20), 1000,
                     required_converged=min(100, n // 10))
    kw = {}
    if kind < 0.45:
        kw["lbfgs_m"] = rng.randint(3, 8)
    if rng.random() < 0.3:
        kw.update(precision="mixed", grad_tol=1e-4)
    n = _log_uniform(rng, 256, _n_max(d, "lbfgs_m" in kw))
    if entry == "host" and n * d < 100000 and "precision" not in kw:
        kw["swarm"] = True
    return _case(None, entry, objective, d, n, rng.randint(0, 20), 1000, **kw)


_KEPT = {}  # what a program makes once: the context, compiled objectives


def _context():
    if "ctx" not in _KEPT:
        _KEPT["ctx"] = Z.zeus_context_create(torch.cuda.current_device())
    return _KEPT["ctx"]


def _source(name):
    return U.ROSENBROCK if name == "rosenbrock" else U.poisson_fit_source()


def _objective(name):
    if name not in _KEPT:
        _KEPT[name] = Z.zeus_objective_compile(_context(), _source(name))
    return _KEPT[name]


_OWN = ("name", "entry", "swarm", "requests", "stream", "n_div", "source")


def _problems(case, seed):
    """The problems of a case (one, or a stream)."""
    if case["entry"] == "batch":
        reqs = W.uneven_batch(case["requests"], seed=case["stream"])
    elif case["entry"] == "served":
        reqs = W.served_mix(case["requests"], seed=case["stream"])
    else:
        return [W.problem(seed=seed, **{k: v for k, v in case.items() if k not in _OWN})]
    return [dict(r, n=max(64, r["n"] // case["n_div"]), seed=seed) for r in reqs]


def prepare(case, seed):
    problems = _problems(case, seed)
    st = {"entry": case["entry"], "ctx": _context(), "problems": [Z.make_problem(p) for p in problems],
          "swarm": bool(case.get("swarm"))}
    if case["entry"] == "device":
        st["solve"] = Z.DeviceSolve(problems[0], pso_state=st["swarm"])
    elif case["entry"] == "plan":
        st["plan"] = Z.DevicePlan(st["ctx"], problems)
    elif case["entry"] == "served":
        if "server" not in _KEPT:
            _KEPT["server"] = Z.Server(st["ctx"], 8 << 30)
        st["server"] = _KEPT["server"]
    elif case["entry"] == "user":
        st["objective"] = _objective(case["source"])
    return st


def _joined(outs):
    """The results of a stream as one array per output, in request order."""
    keys = [k for k in outs[0] if k not in ("summary", "times")]
    res = {k: np.concatenate([o[k].reshape(-1) for o in outs]) for k in keys}
    res["summary"] = {k: np.array([o["summary"][k] for o in outs]) for k in outs[0]["summary"]}
    return res


def run(st):
    entry = st["entry"]
    if entry == "device":
        st["solve"].enqueue(st["ctx"])
        return dict(st["solve"].t)
    if entry == "plan":
        st["plan"].launch()
        return dict(st["plan"].t[0])
    if entry == "host":
        return Z.zeus_minimize(st["ctx"], st["problems"][0], pso_state=st["swarm"])
    if entry == "user":
        return Z.zeus_minimize_user(st["ctx"], st["objective"], st["problems"])[0]
    if entry == "batch":
        return _joined(Z.zeus_minimize_batch(st["ctx"], st["problems"]))
    tickets = [st["server"].submit(p) for p in st["problems"]]
    return _joined([st["server"].wait(t) for t in tickets])


# Steps per start and trials per step that the method takes on these problems
# (means over a few seeds; a solve's own counts come back in its summary).
_STEPS = {"rosenbrock": lambda d: 20 + 5 * d, "rastrigin": lambda d: 14, "ackley": lambda d: 21,
          "styblinski_tang": lambda d: 12, "goldstein_price": lambda d: 12}
_TRIALS = {"rosenbrock": 2.8, "rastrigin": 5.6, "ackley": 1.7, "styblinski_tang": 2.5,
           "goldstein_price": 3.0}
# flops of a term's value and of its tangent
_TERM = {"rosenbrock": (8, 10), "rastrigin": (6, 5), "ackley": (7, 6), "styblinski_tang": (7, 6),
         "goldstein_price": (45, 60)}


def _solve_work(p, source=None):
    d, n = p["dim"], p["n"]
    obj = p["objective"]
    steps, trials, (fv, ft) = 108, 12.2, (40 * 10 / 4, 40 * 14 / 4)  # the likelihood fit: 40 bins
    if obj != "user" or source == "rosenbrock":
        obj = "rosenbrock" if obj == "user" else obj
        steps, trials, (fv, ft) = _STEPS[obj](d), _TRIALS[obj], _TERM[obj]
    steps = min(steps, p["iter_bfgs"])
    h = 8 * p["lbfgs_m"] * d + 3 * d if p.get("lbfgs_m") else 6 * d * d
    sweep = fv * d + 12 * d
    step = h + (fv + 2 * ft) * d + trials * (fv + 2) * d + 14 * d
    flops = n * (sweep * (p["iter_pso"] + 1) + steps * step)
    return 8.0 * n * d + 28.0 * n, flops  # x, f and the five per-start counts written once


def work(case):
    total = [0.0, 0.0]
    for p in _problems(case, 1):
        for k, v in enumerate(_solve_work(p, case.get("source"))):
            total[k] += v
    return {"bytes": total[0], "flops": total[1]}


# ---- the swarm phase in numpy ------------------------------------------------

def _mul_hi_lo(a, k):
    """128-bit product of uint64 array a and constant k as (high, low)."""
    m32, s = np.uint64(0xFFFFFFFF), np.uint64(32)
    al, ah, kl, kh = a & m32, a >> s, np.uint64(k & 0xFFFFFFFF), np.uint64(k >> 32)
    ll, lh, hl = al * kl, al * kh, ah * kl
    mid = (ll >> s) + (lh & m32) + (hl & m32)
    return ah * kh + (lh >> s) + (hl >> s) + (mid >> s), a * np.uint64(k)


def _uniforms(n, d, t, tag, seed):
    """[n, d] uniforms of sweep t: Philox4x64-10 with counter (block, particle, t, tag)."""
    nb = (d + 3) // 4
    c0 = np.tile(np.arange(nb, dtype=np.uint64), n)
    c1 = np.repeat(np.arange(n, dtype=np.uint64), nb)
    c2, c3 = np.full(n * nb, t, np.uint64), np.full(n * nb, tag, np.uint64)
    k0, k1 = seed, 0
    for _ in range(10):
        h0, l0 = _mul_hi_lo(c0, 0xD2E7470EE14C6C93)
        h1, l1 = _mul_hi_lo(c2, 0xCA5A826395121157)
        c0, c1, c2, c3 = h1 ^ c1 ^ np.uint64(k0), l1, h0 ^ c3 ^ np.uint64(k1), l0
        k0 = (k0 + 0x9E3779B97F4A7C15) % 2**64
        k1 = (k1 + 0xBB67AE8584CAA73B) % 2**64
    words = np.stack([c0, c1, c2, c3], axis=1).reshape(n, 4 * nb)[:, :d]
    return (words >> np.uint64(11)).astype(np.float64) * 2.0**-53


def _value(objective, x):
    d = x.shape[1]
    if objective == "rosenbrock":
        return ((1 - x[:, :-1]) ** 2 + 100 * (x[:, 1:] - x[:, :-1] ** 2) ** 2).sum(axis=1)
    if objective == "rastrigin":
        return 10 * d + (x**2 - 10 * np.cos(2 * np.pi * x)).sum(axis=1)
    if objective == "ackley":
        return (-20 * np.exp(-0.2 * np.sqrt((x**2).sum(axis=1) / d))
                - np.exp(np.cos(2 * np.pi * x).sum(axis=1) / d) + 20 + np.e)
    return 0.5 * (x**4 - 16 * x**2 + 5 * x).sum(axis=1)


def exact(case, seed):
    if not case.get("swarm"):
        return None
    p = _problems(case, seed)[0]
    n, d, lo, hi = p["n"], p["dim"], p["lower"], p["upper"]
    vh = p["v_half"] if p["v_half"] > 0 else hi - lo
    x = lo + _uniforms(n, d, 0, 0, seed) * (hi - lo)
    v = -vh + _uniforms(n, d, 0, 1, seed) * (2 * vh)
    px, pf = x.copy(), _value(p["objective"], x)
    for t in range(1, p["iter_pso"] + 1):
        g = px[np.argmin(pf)]
        v = (p["w"] * v + p["c1"] * _uniforms(n, d, t, 2, seed) * (px - x)
             + p["c2"] * _uniforms(n, d, t, 3, seed) * (g - x))
        x = x + v
        f = _value(p["objective"], x)
        better = f < pf
        pf = np.where(better, f, pf)
        px = np.where(better[:, None], x, px)
    out = dict.fromkeys(("f", "x", "iters", "status", "ls_trials", "skips", "resets", "summary"))
    out.update(seeds=x, pso_v=v, pso_px=px, pso_pf=pf, pso_best_x=px[np.argmin(pf)])
    return out
