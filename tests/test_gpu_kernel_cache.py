"""The on-disk cache of compiled kernels: a damaged entry costs a compile,
never a call."""
import numpy as np
import pytest

from paper_1606_08281_amd import workloads as W

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[gpu case]", *a, flush=True)


def _damage(folder):
    files = list(folder.glob("*.co"))
    assert files
    for f in files:
        f.write_bytes(b"not a code object" * 50)
    return files


@pytest.mark.parametrize("path", ["batch", "requests", "ode"])
def test_damaged_cache_entry(monkeypatch, tmp_path, path):
    """A call whose kernel choice finds a damaged entry: the results it has
    without the entry, and the entry whole again."""
    from paper_1606_08281_amd import lik
    monkeypatch.setenv("LIK_KERNEL_CACHE", str(tmp_path))
    if path == "ode":
        wl = W.erk_workload(5)

        def call(kernel=lik.KERNEL_AUTO):
            return lik.ode_eval(lik.OdeModel(wl["spec"]), wl["theta"], wl["trajectories"],
                                kernel=kernel)[0]
        lik.OdeModel(wl["spec"]).precompile()
    else:
        wl = W.telegraph_workload(n_theta=3, n_traj=2, n_obs=5, n_particles=70)
        net = lik.Network(wl.net.orders, wl.net.stoich)
        kw = dict(obs_kind=wl.obs_kind, observed=wl.observed, sigma=wl.sigma, theta=wl.theta,
                  trajectories=wl.trajectories, n_particles=wl.n_particles, seed=wl.seed)

        def call(kernel=lik.KERNEL_AUTO):
            if path == "requests":
                return lik.eval_requests([dict(net=net, **kw)], kernel=kernel)[0][0]
            return lik.eval_batch(net, kernel=kernel, **kw)["loglik"]
        if path == "requests":
            lik.precompile_requests([net], lik.FP64)
        else:
            net.precompile()
    want = call(lik.KERNEL_GENERIC)
    damaged = _damage(tmp_path)
    _say("damaged cache entry,", path)
    for _ in range(2):
        assert np.array_equal(call(), want)
    assert all(b"gfx950" in f.read_bytes() for f in damaged)
