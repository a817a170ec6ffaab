"""Batches too small to fill the GPU: an interval cut into items of fewer than
64 particles, and the kernel the automatic choice takes, against the oracle
and against the generic kernel.  Event counts, final particle counts and
statuses bit for bit; log-likelihoods to 1e-9 relative (the weights' sum is
the only freedom)."""
import numpy as np
import pytest

from paper_1606_08281_amd import workloads as W
from test_gpu_parity import _gpu, _oracle, _say, assert_parity

pytestmark = pytest.mark.gpu

# around the item sizes 4, 8, 16, 32 and 64, and the largest filter
SIZES = [1, 5, 31, 33, 63, 65, 250, 1000, 4096]


@pytest.mark.parametrize("kernel", [1, 2])
@pytest.mark.parametrize("precision", [0, 1])
def test_split_items(orc, precision, kernel):
    """One filter at a time (the most splitting): every item size and ragged
    last items, both schedules; 150 and more events per particle and interval."""
    wl = W.immigration_death_workload(1, t_obs=[5.0, 10.0, 15.0])
    theta = np.array([[30.0, 0.1]])
    for H in SIZES:
        ref = _oracle(orc, wl, theta=theta, H=H, precision=precision)
        for schedule in (1, 0):
            _say("split items H", H, "precision", precision, "kernel", kernel, "schedule", schedule)
            assert_parity(_gpu(wl, theta=theta, H=H, precision=precision, kernel=kernel,
                               tuning={"schedule": schedule}), ref)


@pytest.mark.parametrize("schedule", [1, 0])
def test_split_items_event_cap(orc, schedule):
    """The event cap reached inside split items: the theta's status."""
    wl = W.immigration_death_workload(1, t_obs=[5.0, 10.0])
    theta = np.array([[30.0, 0.1], [20.0, 0.1]])
    for cap in (1, 63, 64, 150, 400):
        ref = _oracle(orc, wl, theta=theta, H=40, event_cap=cap)
        _say("split items cap", cap, "schedule", schedule)
        assert_parity(_gpu(wl, theta=theta, H=40, event_cap=cap, kernel=2,
                           tuning={"schedule": schedule}), ref)


@pytest.mark.parametrize("precision", [0, 1])
def test_split_items_large_network(orc, precision):
    """Rates and net changes in LDS: stopped lanes take the row without a change."""
    wl = W.random_network_workload(n_theta=3, n_particles=45, n_obs=3)
    _say("split items 20x40 precision", precision)
    ref = _oracle(orc, wl, precision=precision)
    for kernel in (1, 2):
        assert_parity(_gpu(wl, precision=precision, kernel=kernel), ref)


def test_automatic_kernel_choice(monkeypatch, tmp_path):
    """A batch below the compile's threshold: generic without a compiled kernel,
    specialised once one is in the disk cache; the results are the same."""
    from paper_1606_08281_amd import lik
    monkeypatch.setenv("LIK_KERNEL_CACHE", str(tmp_path))
    wl = W.telegraph_workload(n_theta=5, n_traj=2, n_obs=6, n_particles=130)

    def run(net, kernel=lik.KERNEL_AUTO):
        return lik.eval_batch(net, wl.obs_kind, wl.observed, wl.sigma, wl.theta, wl.trajectories,
                              wl.n_particles, wl.seed, aux=True, kernel=kernel)

    net = lik.Network(wl.net.orders, wl.net.stoich)
    before = run(net)
    assert not list(tmp_path.iterdir())
    net.precompile()
    after, fresh = run(net), run(lik.Network(wl.net.orders, wl.net.stoich))
    reqs = [dict(net=net, obs_kind=wl.obs_kind, observed=wl.observed, sigma=wl.sigma,
                 theta=wl.theta, trajectories=wl.trajectories, n_particles=wl.n_particles,
                 seed=wl.seed)]
    one = lik.eval_requests(reqs)[0][0]
    lik.precompile_requests([net])
    two = lik.eval_requests(reqs)[0][0]
    for got in (after, fresh, run(net, lik.KERNEL_GENERIC)):
        for k in before:
            assert np.array_equal(before[k], got[k]), k
    assert np.array_equal(one, before["loglik"]) and np.array_equal(two, before["loglik"])


def test_automatic_kernel_choice_under_capture():
    """A small batch captured by its caller before any kernel was loaded, then
    replayed with eager calls between: no module load inside the capture."""
    import torch
    from paper_1606_08281_amd import lik
    wl = W.telegraph_workload(n_theta=3, n_traj=2, n_obs=5, n_particles=70)
    net = lik.Network(wl.net.orders, wl.net.stoich)
    net.precompile()
    db = lik.DeviceBatch(net, wl.obs_kind, wl.observed, wl.sigma, wl.trajectories, wl.n_theta,
                         wl.n_particles)
    theta = torch.from_numpy(wl.theta).cuda()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        db.run(theta, wl.seed)
    for _ in range(3):
        db.loglik.zero_()
        graph.replay()
        torch.cuda.synchronize()
        replayed = db.loglik.clone()
        eager, _ = db.run(theta, wl.seed)
        torch.cuda.synchronize()
        assert torch.equal(replayed, eager)


def test_flow_launch_near_2_to_32_lanes():
    """A batch whose wavefronts, with any spare one beyond 2^26 - 1, would not
    fit one launch: the same results as few of its filters in the per-interval
    schedule."""
    T = 65535
    rng = np.random.default_rng(3)
    wl = W.immigration_death_workload(1)
    tr = dict(t_obs=np.arange(1, T + 1) * 1.0, y=rng.normal(5.0, 2.0, (T, 1)), t0=0.0,
              x0=np.array([5], np.int32))
    theta = np.exp(rng.normal([-9.0, -9.0], 0.5, (1024, 2)))
    kw = dict(trajectories=[tr], H=5, kernel=1)
    _say("flow launch of 1024 x 65535 items")
    got = _gpu(wl, theta=theta, tuning={"schedule": 1}, **kw)
    some = [0, 511, 1023]
    want = _gpu(wl, theta=theta[some], theta_ids=some, tuning={"schedule": 0}, **kw)
    assert np.array_equal(got["loglik"][some], want["loglik"])
    assert np.all(got["status"] == 0)


def test_long_interval_is_no_stall(monkeypatch):
    """One filter whose interval lasts about twice the flow schedule's limit,
    while its items (of 4 particles, started at different counts) finish one
    after another and every wavefront of the launch is resident: not given up."""
    import time
    orders, stoich = np.array([[1, 0], [0, 1]]), np.array([[-1, 1], [1, -1]])   # X <-> Y
    tr = dict(t_obs=np.array([1.0, 2.0]), y=np.full((2, 1), 2e5), t0=0.0,
              x0=np.array([4000, 0], np.int32), x0_hi=np.array([400000, 0], np.int32))
    from paper_1606_08281_amd import lik
    net = lik.Network(orders, stoich)

    def run():
        return lik.eval_batch(net, lik.OBS_GAUSSIAN, [0], 1e5, np.array([[1.0, 1.0]]), [tr], 4096,
                              7, kernel=lik.KERNEL_GENERIC)
    _say("interval longer than the stall limit: without the limit")
    want = run()
    t = time.perf_counter()
    run()
    limit_us = int((time.perf_counter() - t) * 1e6 / 4)     # half an interval
    monkeypatch.setenv("LIK_FLOW_STALL_US", str(limit_us))
    _say("interval longer than the stall limit of", limit_us, "us")
    got = run()
    assert got["status"][0] == 0 and np.array_equal(got["loglik"], want["loglik"])


def _three_species_workload():
    """26 reactions of 3 species: births, deaths, conversions and pairs, each
    several times (few species: pools of up to 6 groups fit)."""
    kinds = [({}, {0: 1}, 20.0), ({}, {1: 1}, 10.0), ({0: 1}, {0: -1}, 0.3),
             ({1: 1}, {1: -1, 2: 1}, 0.3), ({2: 1}, {2: -1}, 0.3), ({2: 1}, {2: -1, 0: 1}, 0.2),
             ({0: 1, 1: 1}, {0: -1}, 0.002), ({1: 2}, {1: -2, 2: 1}, 0.002)]
    orders, stoich = np.zeros((26, 3), np.int32), np.zeros((26, 3), np.int32)
    rates = np.zeros(26)
    for r in range(26):
        p, v, rates[r] = kinds[r % len(kinds)]
        for u, k in p.items():
            orders[r, u] = k
        for u, k in v.items():
            stoich[r, u] = k
    rng = np.random.default_rng(2)
    t = np.array([1.0, 2.0, 3.0])
    tr = {"t_obs": t, "y": rng.normal(60.0, 10.0, (3, 1)), "t0": 0.0,
          "x0": np.array([40, 30, 50], np.int32)}
    theta = rates * np.exp(rng.normal(0.0, 0.3, (512, 26)))
    net = W.Network("3x26", ["A", "B", "C"], orders, stoich)
    return W.Workload("3x26", net, 0, [0], 10.0, theta, [tr], 200)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("network", ["20x40", "3x26"])
def test_event_cap_in_the_branch_free_main_loop(orc, network, precision):
    """More than 24 reactions, whole groups of 64 (too many of them to be split);
    3 species: pools whose lanes take further particles.  The cap before, on and
    after the second event of a random block in FP32-mixed."""
    if network == "3x26":
        wl, caps = _three_species_workload(), (1, 281, 310, 311, 330, 331, 345, 400)
    else:
        wl = W.random_network_workload(n_theta=512, n_particles=200, n_obs=3)
        caps = (1, 301, 600, 601, 700, 701, 801, 1000)
    idx = np.arange(5, 512, 73)
    capped = 0
    for cap in caps:
        ref = _oracle(orc, wl, theta=wl.theta[idx], theta_ids=idx, precision=precision,
                      event_cap=cap)
        capped += int((ref["status"] == 1).sum())
        for kernel, pool_min in ((1, 1), (2, 1), (2, 4)):
            _say(network, "cap", cap, "precision", precision, "kernel", kernel, "pool", pool_min)
            got = _gpu(wl, precision=precision, kernel=kernel, event_cap=cap,
                       tuning={"schedule": 0, "pool_min": pool_min, "pool_max": 6,
                               "items_per_cu": 0})
            assert np.array_equal(got["status"][idx], ref["status"])
            assert np.array_equal(np.isnan(got["loglik"][idx]), np.isnan(ref["loglik"]))
            ok = ref["status"] == 0
            assert np.array_equal(got["filter_events"][idx][ok], ref["events"][ok])
            assert np.array_equal(got["final_state"][idx][ok], ref["final_state"][ok])
    assert 0 < capped < len(caps) * len(idx)


@pytest.mark.parametrize("kernel", [1, 2])
def test_split_filters_that_wait(kernel):
    """Hundreds of filters with uneven chains under a short queue: filters are
    split while others are parked, and more would be split than the launch has
    wavefronts or ring room for.  The per-interval schedule's results."""
    rng = np.random.default_rng(11)
    wl = W.immigration_death_workload(1, t_obs=5.0 * np.arange(1, 9))
    for H, n in ((150, 350), (64, 1500), (1000, 40)):
        theta = np.exp(rng.normal([3.0, -2.0], [1.0, 0.3], (n, 2)))
        want = _gpu(wl, theta=theta, H=H, kernel=kernel, tuning={"schedule": 0})
        for urgent in (0, 1 << 30):
            _say("split and parked filters H", H, "filters", n, "urgent", urgent)
            got = _gpu(wl, theta=theta, H=H, kernel=kernel,
                       tuning={"schedule": 1, "backlog_per_cu": 1, "urgent_events": urgent})
            for k in ("loglik", "status", "filter_events", "final_state"):
                assert np.array_equal(got[k], want[k], equal_nan=True), k
