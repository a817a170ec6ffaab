"""The two specialised ODE kernels -- a group of lanes per (theta, trajectory)
pair for small populations, a lane per pair for large ones -- take the same
operations in the same order: equal results, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[gpu case]", *a, flush=True)


@pytest.mark.parametrize("n_species", [1, 16, 17, 32])
def test_group_and_wide_kernels_agree(n_species):
    """The kernel of small populations (a group of lanes per pair: 16 up to 16
    species, 32 above) against the one of large ones (a lane per pair) and the
    generic one: chains of decays with every factor kind, equal results and
    step counts, ragged last workgroups."""
    from paper_1606_08281_amd import lik
    U = n_species
    terms = [{"to": 0, "rate_param": 0, "factors": []}]
    for s in range(U):
        to = {"to": s + 1} if s + 1 < U else {}
        terms.append(dict(frm=s, rate_param=1, factors=[(s % 4, s, 2)], **to))
    spec = {"U": U, "V": 3, "terms": terms, "x0_param": [-1] * U, "obs_kind": 0,
            "obs_species": U - 1, "sd_param": -1, "sd_const": 0.5}
    model = lik.OdeModel(spec)
    rng = np.random.default_rng(U)
    t = np.array([0.3, 0.9, 1.0])
    trajs = [{"t_obs": t, "y": rng.normal(1.0, 0.3, 3), "x0": np.linspace(1.0, 2.0, U)}]
    n = 49153 + 5   # one lane per pair; in parts, groups
    theta = np.exp(rng.normal(0.0, 0.5, (n, 3)))
    theta[7, 1] = -1.0
    _say("group and wide ODE kernels, species", U)
    wide = lik.ode_eval(model, theta, trajs, steps=True)
    for lo, hi in ((0, 1), (1, 4), (4, 1004), (n - 1003, n)):
        for kernel in (lik.KERNEL_GENERIC, lik.KERNEL_SPECIALIZED):
            part = lik.ode_eval(model, theta[lo:hi], trajs, steps=True, kernel=kernel)
            for a, b in zip(part, wide):
                assert np.array_equal(a, b[lo:hi], equal_nan=True)
