"""Performance cases: likelihood evaluations as programs ask for them, through the public entry points.

Callers of this library are samplers: they propose rate vectors and want the
log-likelihood of each.  The cases run from one rate vector (an interactive
call, the shortest chain of launches) over a sampler's proposal batches, the
served and the many-request paths, to whole populations that fill the GPU;
both precisions, every observation model, small and large networks, and the
deterministic model.  `draw` spreads the same kinds of call over their ranges.

Sizes are those of the repository's own workloads, benchmark and serving mixes.
"""
import functools
import math

import numpy as np
import torch

from paper_1606_08281_amd import lik
from paper_1606_08281_amd import workloads as W

PRECISION = {"fp64": lik.FP64, "mixed": lik.FP32_MIXED}
KERNEL = {"auto": lik.KERNEL_AUTO, "specialized": lik.KERNEL_SPECIALIZED}

# Direct-method events per particle and observation interval of each model at
# its prior (measured over whole batches): the size of the work, not its bound.
EVENTS = {"immigration_death": 104, "telegraph": 115, "lacgfp": 6600, "random_long": 11700,
          "random_light": 36}
REACTIONS = {"immigration_death": 2, "telegraph": 6, "lacgfp": 18, "random_long": 40,
             "random_light": 40}
ODE_ATTEMPTS = 454       # step attempts per (parameter vector, input pattern)
ODE_OPERATIONS = 1450    # binary64 operations of one attempt


def _stochastic(name, api, model, thetas, trajectories, observations, particles, precision="fp64",
                kernel="auto"):
    return {"name": name, "api": api, "model": model, "thetas": thetas,
            "trajectories": trajectories, "observations": observations, "particles": particles,
            "precision": precision, "kernel": kernel}


def listed():
    return [
        # One rate vector, one trajectory, few particles: a call from an
        # interactive session; launches and the chain of intervals are all of it.
        _stochastic("single_theta", "device", "immigration_death", 1, 1, 20, 100),
        # A proposal round of the level-set sampler: a few rate vectors that
        # survived the rejection step, three trajectories.
        _stochastic("proposal_round", "device", "telegraph", 13, 3, 50, 512),
        # The birth-death example's whole prior sample from host arrays.
        _stochastic("host_batch", "host", "immigration_death", 64, 1, 20, 256),
        # A population of the gene-expression model (the benchmark batch).
        _stochastic("telegraph_population", "device", "telegraph", 1024, 10, 50, 1000),
        # The same model in the cheaper precision, half the population.
        _stochastic("telegraph_mixed", "device", "telegraph", 512, 10, 50, 1000, "mixed"),
        # The 18-reaction model: random initial counts, fluorescence read-out,
        # particles that differ by orders of magnitude in events.
        _stochastic("lacgfp_population", "device", "lacgfp", 256, 5, 29, 200),
        # A large network over long intervals (the SSA alone counts) ...
        _stochastic("random_long", "device", "random_long", 512, 1, 16, 512),
        # ... and over short ones (hand-offs and weighing count as well).
        _stochastic("random_light_mixed", "device", "random_light", 250, 1, 100, 512, "mixed"),
        # Many single-vector requests of two models, uneven lengths and
        # particle counts, evaluated in one call.
        {"name": "uneven_requests", "api": "requests", "requests": 512, "longest": 200,
         "precision": "fp64"},
        # Requests of three models submitted to the server together.
        {"name": "served_mix", "api": "server", "requests": 48, "longest": 50,
         "precision": "fp64"},
        # The deterministic model: a whole population resident on the GPU ...
        {"name": "erk_population", "api": "ode_device", "thetas": 65536, "observations": 60},
        # ... and one sampler batch from host arrays.
        {"name": "erk_batch", "api": "ode_host", "thetas": 200, "observations": 60},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["immigration_death", "telegraph", "telegraph", "lacgfp", "random_long",
                       "random_light", "requests", "server", "ode"])
    precision = rng.choice(["fp64", "fp64", "mixed"])
    api = rng.choice(["device", "device", "host"])
    if kind == "immigration_death":
        return _drawn(api, kind, _log_int(rng, 1, 300), 1, rng.randint(5, 60),
                      _log_int(rng, 40, 4096), precision)
    if kind == "telegraph":
        return _drawn(api, kind, _log_int(rng, 1, 700), rng.randint(1, 10), rng.randint(5, 50),
                      _log_int(rng, 60, 1100), precision, rng.choice(["auto", "specialized"]))
    if kind == "lacgfp":
        return _drawn(api, kind, _log_int(rng, 4, 200), rng.randint(1, 5), rng.randint(4, 29),
                      _log_int(rng, 50, 220), precision, "specialized")
    if kind == "random_long":
        return _drawn(api, kind, _log_int(rng, 8, 256), 1, rng.randint(2, 12),
                      _log_int(rng, 100, 600), precision, "specialized")
    if kind == "random_light":
        return _drawn(api, kind, _log_int(rng, 2, 600), 1, rng.randint(10, 100),
                      _log_int(rng, 100, 1000), precision)
    if kind == "requests":
        return {"api": kind, "requests": _log_int(rng, 8, 600), "longest": rng.randint(20, 200),
                "precision": precision}
    if kind == "server":
        return {"api": kind, "requests": _log_int(rng, 1, 60), "longest": rng.randint(12, 50),
                "precision": precision}
    return {"api": rng.choice(["ode_device", "ode_host"]), "thetas": _log_int(rng, 1, 60000),
            "observations": rng.randint(20, 60)}


def _drawn(*args):
    case = _stochastic("", *args)
    del case["name"]
    return case


# -- inputs -------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _paths(model, observations):
    """The workload a model's noise-free observation paths come from."""
    if model == "immigration_death":
        return W.immigration_death_workload(1, t_obs=5.0 * np.arange(1, observations + 1))
    if model == "telegraph":
        return W.telegraph_workload(1, n_traj=10, n_obs=observations)
    if model == "lacgfp":
        return W.lacgfp_workload(theta=W.LACGFP_TRUTH, n_traj=5, n_obs=29)
    if model == "random_long":
        return W.random_network_workload(1, n_obs=16, dt=W.RANDOM_DT_1E4)
    return W.random_network_workload(512, n_obs=100)


def _trajectories(model, count, observations, rng):
    """`count` observed trajectories: the model's paths with fresh measurement noise."""
    longest = {"immigration_death": 200, "telegraph": 200 if observations > 50 else 50}
    wl = _paths(model, longest.get(model, 0))
    out = []
    for tr in wl.trajectories[:count]:
        tr = dict(tr, t_obs=tr["t_obs"][:observations])
        x = tr.pop("x_true")[:observations].astype(np.float64)
        if model == "immigration_death":
            y = x + rng.normal(0.0, 2.0, x.shape)
        elif model == "telegraph":
            y = x[:, 3:4] * np.exp(rng.normal(0.0, 0.1, (observations, 1)))
        elif model == "lacgfp":
            mature = x[:, 8:9]
            y = (rng.normal(W.LACGFP_GAIN * mature, W.LACGFP_SD * np.sqrt(mature))
                 + rng.normal(W.LACGFP_BG_MEAN, W.LACGFP_BG_SD, mature.shape))
        else:
            y = x[:, :2] + rng.normal(0.0, 10.0, (observations, 2))
        tr["y"] = y
        tr.pop("x0_drawn", None)
        out.append(tr)
    return wl, out


def _rates(model, count, rng):
    """`count` rate vectors: prior draws (Lac-Gfp: a late level's population)."""
    if model == "immigration_death":
        return W.log_uniform(rng, [1e-2, 1e-2], [1e2, 1e2], count)
    if model == "telegraph":
        return W.log_uniform(rng, W.TELEGRAPH_TRUTH / 10, W.TELEGRAPH_TRUTH * 10, count)
    if model == "lacgfp":
        spread = np.exp(rng.normal(0.0, 0.3, (count, len(W.LACGFP_TRUTH))))
        return W.lacgfp_rates(W.LACGFP_TRUTH * spread)
    return W.log_uniform(rng, np.full(40, 1e-3), np.full(40, 1.0), count)


@functools.lru_cache(maxsize=None)
def _network(model):
    """A program keeps its network for every call."""
    wl = _paths(model, {"immigration_death": 200, "telegraph": 50}.get(model, 0))
    return lik.Network(wl.net.orders, wl.net.stoich)


@functools.lru_cache(maxsize=None)
def _compiled(models, precision):
    """A program that calls again and again compiles its kernels ahead, once."""
    nets = [_network(m) for m in models]
    for net in nets:
        net.precompile(PRECISION[precision])
    if len(nets) > 1:
        lik.precompile_requests(nets, PRECISION[precision])


@functools.lru_cache(maxsize=None)
def _server():
    return lik.Server()


@functools.lru_cache(maxsize=None)
def _ode():
    wl = W.erk_workload(1)
    return wl["spec"], wl["trajectories"], lik.OdeModel(wl["spec"])


def _rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def _ode_inputs(case, seed):
    rng = _rng(seed)
    spec, base, model = _ode()
    n = case["observations"]
    trajectories = []
    for tr in base:
        noise = rng.normal(0.0, 0.01, n) - rng.normal(0.0, 0.01, n)
        trajectories.append({"t_obs": tr["t_obs"][:n], "y": tr["y"][:n] + noise, "t0": tr["t0"],
                             "x0": tr["x0"], "t_in": tr["t_in"], "u_in": tr["u_in"]})
    spread = np.exp(rng.normal(0.0, 0.3, (case["thetas"], len(W.ERK_REF))))
    return spec, model, trajectories, W.erk_engine_params(W.ERK_REF * spread)


def _request(model, thetas, trajectories, observations, particles, precision, rng):
    wl, trs = _trajectories(model, trajectories, observations, rng)
    return {"net": _network(model), "obs_kind": wl.obs_kind, "observed": wl.observed,
            "sigma": wl.sigma, "theta": _rates(model, thetas, rng), "trajectories": trs,
            "n_particles": particles, "seed": int(rng.integers(1 << 62)),
            "precision": PRECISION[precision]}


UNEVEN = ("immigration_death", "telegraph")
MIX_SIZES = 13   # the stream of request sizes, the same for every set of inputs


def _requests(case, seed):
    """The uneven batch: one rate vector each, two models in turn, 10 or more observations."""
    rng, sizes = _rng(seed), _rng(MIX_SIZES)
    return [_request(UNEVEN[k % 2], 1, 1, int(sizes.integers(10, case["longest"] + 1)),
                     int(sizes.choice([128, 512, 1024, 4096])), case["precision"], rng)
            for k in range(case["requests"])]


def _served(case, seed):
    """The serving mix: 60 % telegraph, 20 % immigration-death, 20 % the large network."""
    rng, sizes = _rng(seed), _rng(MIX_SIZES)
    out = []
    for _ in range(case["requests"]):
        u = sizes.random()
        model = "telegraph" if u < 0.6 else "immigration_death" if u < 0.8 else "random_light"
        large = model == "random_light"
        out.append(_request(model, int(sizes.integers(1, 9 if large else 33)),
                            int(sizes.integers(1, 4)) if model == "telegraph" else 1,
                            100 if large else int(sizes.integers(10, case["longest"] + 1)),
                            512 if large else int(sizes.choice([128, 512, 1000])),
                            case["precision"], rng))
    return out


def prepare(case, seed):
    api = case["api"]
    if api == "requests":
        _compiled(UNEVEN, case["precision"])
        return {"api": api, "requests": _requests(case, seed)}
    if api == "server":
        return {"api": api, "server": _server(), "requests": _served(case, seed)}
    if api in ("ode_device", "ode_host"):
        _, model, trajectories, theta = _ode_inputs(case, seed)
        if api == "ode_host":
            return {"api": api, "model": model, "theta": theta, "trajectories": trajectories}
        return {"api": api, "theta": torch.from_numpy(theta).cuda(),
                "batch": lik.OdeDeviceBatch(model, trajectories, len(theta), steps=True)}
    _compiled((case["model"],), case["precision"])
    kernel = KERNEL[case["kernel"]]
    q = _request(case["model"], case["thetas"], case["trajectories"], case["observations"],
                 case["particles"], case["precision"], _rng(seed))
    if api == "host":
        return {"api": api, "request": dict(q, kernel=kernel)}
    batch = lik.DeviceBatch(q["net"], q["obs_kind"], q["observed"], q["sigma"], q["trajectories"],
                            len(q["theta"]), q["n_particles"], precision=q["precision"],
                            kernel=kernel)
    return {"api": api, "batch": batch, "theta": torch.from_numpy(q["theta"]).cuda(),
            "seed": q["seed"]}


def run(state):
    api = state["api"]
    if api == "device":
        batch = state["batch"]
        loglik, status = batch.run(state["theta"], state["seed"])
        return {"loglik": loglik, "status": status, "events": batch.events,
                "filter_loglik": batch.filter_loglik}
    if api == "host":
        return lik.eval_batch(**state["request"], aux=True)
    if api == "requests":
        loglik, status, _ = lik.eval_requests(state["requests"])
        return {"loglik": np.concatenate(loglik), "status": np.concatenate(status)}
    if api == "server":
        server = state["server"]
        tickets = [server.submit(**q) for q in state["requests"]]
        done = [server.wait(t) for t in tickets]
        return {"loglik": np.concatenate([d[0] for d in done]),
                "status": np.concatenate([d[1] for d in done])}
    if api == "ode_device":
        batch = state["batch"]
        loglik, status = batch.run(state["theta"])
        return {"loglik": loglik, "status": status, "steps": batch.steps}
    loglik, status, steps = lik.ode_eval(state["model"], state["theta"], state["trajectories"],
                                         steps=True)
    return {"loglik": loglik, "status": status, "steps": steps}


def work(case):
    """Rates and data in, log-likelihoods, statuses and event counts out; the
    operations of the events (random block, logarithm, quotient, propensities,
    choice of the reaction) or of the solver's step attempts."""
    api = case["api"]
    if api in ("ode_device", "ode_host"):
        pairs = 6 * case["thetas"]
        return {"bytes": case["thetas"] * (36 * 8 + 12) + pairs * 4 + 6 * case["observations"] * 16,
                "flops": pairs * (case["observations"] / 60) * ODE_ATTEMPTS * ODE_OPERATIONS}
    if api in ("requests", "server"):
        n, t = case["requests"], (10 + case["longest"]) / 2
        if api == "requests":
            mix = [("immigration_death", 0.5, 1, 1440 * t), ("telegraph", 0.5, 1, 1440 * t)]
        else:
            mix = [("telegraph", 0.6, 16.5, 2 * 547 * t), ("immigration_death", 0.2, 16.5, 547 * t),
                   ("random_light", 0.2, 4.5, 512 * 100)]
        flops = sum(n * share * thetas * steps * EVENTS[m] * _operations(m, case["precision"])
                    for m, share, thetas, steps in mix)
        return {"bytes": sum(n * s * (k * (REACTIONS[m] * 8 + 12) + 16 * t) for m, s, k, _ in mix),
                "flops": flops}
    m, filters = case["model"], case["thetas"] * case["trajectories"]
    events = filters * case["particles"] * case["observations"] * EVENTS[m]
    return {"bytes": case["thetas"] * (REACTIONS[m] * 8 + 12) + 16 * filters
            + 16 * case["trajectories"] * case["observations"],
            "flops": events * _operations(m, case["precision"])}


def _operations(model, precision):
    """Lane operations of one event: 3 per reaction for its propensity, 2 for
    the choice, and the draw, which costs less in the mixed precision."""
    return (110 if precision == "fp64" else 70) + 5 * REACTIONS[model]


# -- reference values ---------------------------------------------------------

def exact(case, seed):
    """What run() returns, by the documented method in numpy's binary64: the
    particle filter for immigration-death batches (other networks take minutes
    in numpy), the Dormand-Prince solution for deterministic batches of up to
    2,000 trajectories."""
    api = case["api"]
    if api in ("ode_device", "ode_host"):
        if case["thetas"] > 330:
            return None
        spec, _, trajectories, theta = _ode_inputs(case, seed)
        return {"loglik": _ode_exact(spec, theta, trajectories), "status": None, "steps": None}
    if api not in ("device", "host") or case["model"] != "immigration_death" \
            or case["precision"] != "fp64" \
            or case["thetas"] * case["particles"] * case["observations"] > 400_000:
        return None
    q = _request(case["model"], case["thetas"], case["trajectories"], case["observations"],
                 case["particles"], case["precision"], _rng(seed))
    ll = np.array([_filter_exact(c, i, q["trajectories"][0], q["n_particles"], q["seed"], q["sigma"])
                   for i, c in enumerate(q["theta"])])
    out = {"loglik": ll, "status": None}
    if api == "host":
        return out | {"filter_events": None, "filter_loglik": ll, "final_state": None}
    return out | {"events": None, "filter_loglik": ll}


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 over arrays of counters; four arrays of 32-bit words."""
    c0, c1, c2, c3 = (np.asarray(c, dtype=np.uint64) for c in np.broadcast_arrays(c0, c1, c2, c3))
    low, shift = np.uint64(0xFFFFFFFF), np.uint64(32)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = c0 * np.uint64(0xD2511F53), c2 * np.uint64(0xCD9E8D57)
        c0, c1, c2, c3 = ((p1 >> shift) ^ c1 ^ np.uint64(k0), p1 & low,
                          (p0 >> shift) ^ c3 ^ np.uint64(k1), p0 & low)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def _draws(n0, count, j, interval, theta_id, seed):
    """-log u1 and u2 of events n0 .. n0 + count - 1 of the particles j."""
    w0, w1, w2, w3 = _philox(np.arange(n0, n0 + count, dtype=np.uint64)[:, None],
                             j.astype(np.uint64)[None, :], interval, theta_id << 2, seed)
    high, cut = np.uint64(32), np.uint64(11)
    u1 = (((w1 << high) | w0) >> cut).astype(np.float64) * 2.0 ** -53 + 2.0 ** -53
    return -np.log(u1), (((w3 << high) | w2) >> cut).astype(np.float64) * 2.0 ** -53


def _filter_exact(c, theta_id, traj, particles, seed, sigma):
    """log p(y | c) of the immigration-death model by the bootstrap filter:
    direct-method paths, normal weights, systematic resampling in 2^-32 units."""
    x = np.full(particles, float(traj["x0"][0]))
    ll, start = 0.0, float(traj["t0"])
    for t, (end, y) in enumerate(zip(traj["t_obs"], traj["y"][:, 0])):
        if t:
            w0, w1, _, _ = _philox(0, 0, t, (theta_id << 2) | 1, seed)
            q = [int(v) for v in np.floor(e * 2.0 ** 32)]
            total = sum(q)
            rho = (((int(w1) << 32) | int(w0)) * total) >> 64
            ends = particles * np.cumsum(np.array(q, dtype=object))
            points = np.array([k * total + rho for k in range(particles)], dtype=object)
            x = x[np.searchsorted(ends, points, side="right")]
        j, xs, clock, n, chunk = np.arange(particles), x.copy(), np.full(particles, start), 0, 64
        while len(j):
            nl, u2 = _draws(n, chunk, j, t, theta_id, seed)
            live = np.ones(len(j), dtype=bool)
            for k in range(chunk):
                s = c[0] + c[1] * xs
                with np.errstate(divide="ignore"):
                    tau = np.where(s > 0.0, nl[k] / s, np.inf)
                live &= ~(clock + tau > end)
                clock = np.where(live, clock + tau, clock)
                xs = np.where(live, np.where(c[0] > u2[k] * s, xs + 1.0, xs - 1.0), xs)
                if not live.any():
                    break
            x[j[~live]] = xs[~live]
            j, xs, clock, n = j[live], xs[live], clock[live], n + chunk
        l = -0.5 * ((y - x) / sigma) ** 2
        e = np.exp(l - l.max())
        ll += l.max() + math.log(e.sum()) - math.log(particles) \
            - math.log(sigma) - 0.5 * math.log(2.0 * math.pi)
        start = end
    return ll


_A = [[], [1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
      [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
      [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
      [35 / 384, 0.0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]]
_E = [71 / 57600, 0.0, -71 / 16695, 71 / 1920, -17253 / 339200, 22 / 525, -1 / 40]


def _combine(weights, stages):
    total = None
    for a, k in zip(weights, stages):
        if a:
            total = a * k if total is None else total + a * k
    return total


def _ode_rhs(spec, th, u, x):
    dx = np.zeros_like(x)
    for term in spec["terms"]:
        v = np.full(x.shape[1], float(term.get("rate_scale", 1.0)))
        if term.get("rate_param", -1) >= 0:
            v = v * th[term["rate_param"]]
        for kind, sp, par in term.get("factors", []):
            xs, K = x[sp], th[par]
            v = v * (u if kind == 4 else xs if kind == 0 else xs / (K + xs) if kind == 1
                     else xs * xs / (K + xs * xs) if kind == 2 else K / (K + xs * xs))
        if term.get("frm", -1) >= 0:
            dx[term["frm"]] -= v
        if term.get("to", -1) >= 0:
            dx[term["to"]] += v
    return dx


def _ode_exact(spec, theta, trajectories, rtol=1e-6, atol=1e-9):
    """Per parameter vector, the summed normal log-density of the FRET
    observations around the solution (Dormand-Prince 5(4), steps ending at
    every observation and input breakpoint)."""
    th = theta.T
    loglik = np.zeros(th.shape[1])
    lam, bg, E, fAA, fDD = (th[k] for k in spec["fret_param"])
    sd = th[spec["sd_param"]]
    for tr in trajectories:
        t0, t_obs = float(tr["t0"]), tr["t_obs"]
        x = np.repeat(np.asarray(tr["x0"], dtype=np.float64)[:, None], th.shape[1], axis=1)
        for s, p in enumerate(spec["x0_param"]):
            if p >= 0:
                x[s] = th[p]
        stops = [(t, 0, k) for k, t in enumerate(t_obs)]
        stops += [(t, 1, k) for k, t in enumerate(tr["t_in"]) if t0 < t < t_obs[-1]]
        before = [k for k, t in enumerate(tr["t_in"]) if t <= t0]
        u = tr["u_in"][before[-1]] if before else 0.0
        t_now, h = t0, np.full(th.shape[1], 0.01 * (t_obs[0] - t0))
        k1 = _ode_rhs(spec, th, u, x)
        for stop, is_input, k in sorted(stops, key=lambda v: (v[0], v[1])):
            t = np.full(th.shape[1], t_now)
            run_ = np.nonzero(t < stop)[0]
            while len(run_):
                last = t[run_] + h[run_] >= stop
                hs = np.where(last, stop - t[run_], h[run_])
                par, x0, ks = th[:, run_], x[:, run_], [k1[:, run_]]
                for row in _A[1:]:
                    new = x0 + hs * _combine(row, ks)
                    ks.append(_ode_rhs(spec, par, u, new))
                scale = atol + rtol * np.maximum(np.abs(x0), np.abs(new))
                err = (np.abs(hs * _combine(_E, ks)) / scale).max(axis=0)
                with np.errstate(divide="ignore"):
                    h[run_] = hs * np.clip(0.9 * err ** -0.2, 0.2, 5.0)
                ok = err <= 1.0
                moved = run_[ok]
                t[moved] = np.where(last, stop, t[run_] + hs)[ok]
                x[:, moved], k1[:, moved] = new[:, ok], ks[6][:, ok]
                run_ = run_[t[run_] < stop]
            t_now = stop
            if is_input:
                u = tr["u_in"][k]
                k1 = _ode_rhs(spec, th, u, x)
                continue
            a, b = x[spec["obs_species"]], x[spec["obs_species2"]]
            g = lam * (E * fAA * a / ((b + (1.0 - E) * a) * fDD) + bg)
            z = (tr["y"][k] - g) / sd
            loglik += -0.5 * z * z - (np.log(sd) + 0.5 * math.log(2.0 * math.pi))
    return loglik
