"""What the host side plans before it launches, without a GPU: workspace
sizes, and the kernel launches of a call, recorded by a program that answers
the HIP runtime's calls itself (helpers/launch_probe.cpp)."""
import os
import subprocess

import numpy as np
import pytest

from paper_1606_08281_amd import lik


def _network(U):
    orders, stoich = np.zeros((1, U), np.int32), np.zeros((1, U), np.int32)
    stoich[0, 0] = 1
    return lik.Network(orders, stoich)


# (species, particles) -> filters that fit the no-allocation entry point's 64 MiB
SCRATCH_FITS = {(1, 200): 8729, (4, 1000): 1232, (4, 200): 4859, (9, 65): 5526, (20, 64): 5670,
                (32, 64): 3734, (32, 4096): 59}


@pytest.mark.parametrize("shape", sorted(SCRATCH_FITS))
def test_workspace_size_never_shrinks_with_the_batch(shape):
    """A workspace made for a batch holds every smaller one, and the largest
    batch of the no-allocation entry point stays what it was."""
    U, H = shape
    net, size = _network(U), lik.lib().lik_workspace_size
    need = [size(net.handle, n, 1, H) for n in range(9000)]
    shrinks = [n for n in range(1, 9000) if need[n] < need[n - 1]]
    assert not shrinks
    assert sum(b <= 64 << 20 for b in need) - 1 == SCRATCH_FITS[shape]


HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """launches(*args): the calls' kernel launches, [(name, blocks, threads, stream)]."""
    from paper_1606_08281_amd import build
    exe = str(tmp_path_factory.mktemp("probe") / "launch_probe")
    folder = os.path.dirname(os.path.abspath(lik.LIB_PATH))
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I/opt/rocm/include", "-o", exe,
                    os.path.join(HERE, "helpers", "launch_probe.cpp"), f"-L{folder}",
                    "-l:liblik.so", f"-Wl,-rpath,{folder}:{build.hip_runtime_dir()}",
                    "-Wl,--allow-shlib-undefined", "-ldl"], check=True)

    def run(*args, raw=False):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True)
        rows = [line.split() for line in out.stdout.splitlines()]
        return rows if raw else [(r[0], int(r[1]), int(r[2]), r[3]) for r in rows]
    return run


@pytest.mark.parametrize("entry", ["batch", "requests"])
@pytest.mark.parametrize("filters,intervals", [(1, 20), (1024, 64511), (1024, 64512),
                                               (1024, 65535), (4095, 16388)])
def test_flow_launch_stays_below_2_to_32_lanes(launches, entry, filters, intervals):
    """One wavefront per group of 64 particles of every interval, and spare
    ones as far as a launch takes them (fewer than 2^32 lanes): up to, at and
    beyond 2^26 - 2^20 groups."""
    items = filters * intervals
    assert items < 1 << 26
    flow = [r for r in launches(entry, filters, intervals, 64, 1)
            if r[0] in ("k_flow", "k_flow_multi")]
    assert len(flow) == 1
    _, blocks, threads, _ = flow[0]
    assert threads == 64 and items <= blocks and blocks * threads < 1 << 32
    # spare wavefronts: for every interval in items of 4 particles, at most 2^20
    assert blocks == items + min(15 * items, 1 << 20, (1 << 26) - 1 - items)


@pytest.mark.parametrize("entry", ["batch", "requests"])
def test_more_groups_take_the_per_interval_schedule(launches, entry):
    names = [r[0] for r in launches(entry, 8192, 1024, 512, 1)]   # 2^26 groups
    assert "k_flow" not in names and "k_flow_multi" not in names
    assert names.count("k_propagate") == 1024


@pytest.mark.parametrize("failing", [-1, 0, 1, 2, 3])
def test_groups_beside_each_other_are_always_waited_for(launches, failing):
    """The server's iteration over four groups: its stream waits for every
    stream that ran one, also when a group's launch fails; the next admission on
    it may reuse the slots and memory of a finished request."""
    rows = launches("groups", 4, failing, raw=True)
    used = {r[3] for r in rows if r[0] == "k_propagate"} - {"0x10"}
    waited = {r[2] for r in rows if r[0] == "wait" and r[1] == "0x10"}
    assert used <= waited
    assert (rows[-1] == ["returned", "0"]) == (failing < 0)
    assert any(r[0] == "k_weigh" for r in rows) == (failing < 0)
    if failing < 0:
        assert used == {"0x100", "0x200"}


@pytest.mark.parametrize("entry,admit", [("batch", "k_admit"), ("requests", "k_admit_requests")])
def test_ordering_sums_are_cleared_before_the_admission(launches, entry, admit):
    """The admission adds its estimates to the first interval's sum of expected
    events; clearing the sums after it would throw them away (and leave it
    adding to memory that nothing has set)."""
    names = [r[0] for r in launches(entry, 4, 3, 64, 0)]
    assert names.count("k_order_reset") == 1
    assert names.index("k_order_reset") < names.index(admit) < names.index("k_order_count")
    assert "k_order_reset" not in [r[0] for r in launches(entry, 4, 3, 64, 1)]


@pytest.mark.parametrize("entry,generic,cached", [("batch", "k_flow", "lik_flow_spec"),
                                                  ("requests", "k_flow_multi",
                                                   "lik_flow_spec_multi")])
def test_automatic_choice_takes_the_cached_kernel(launches, entry, generic, cached, monkeypatch,
                                                  tmp_path):
    """A batch too small to pay for a compile: the specialised kernel where the
    disk cache of the moment of the call holds it, else the generic one, and
    nothing is compiled."""
    full, empty = tmp_path / "full", tmp_path / "empty"
    empty.mkdir()
    monkeypatch.setenv("LIK_KERNEL_CACHE", str(full))
    net = lik.Network(np.array([[0], [1]]), np.array([[1], [-1]]))   # the probe's network
    net.precompile()
    lik.precompile_requests([net], lik.FP64)

    def kernels(kernel, *folders):
        return [r[0] for r in launches(entry, 4, 3, 64, 1, kernel, *folders)
                if r[0] in (generic, cached)]
    assert kernels(lik.KERNEL_AUTO, empty) == [generic]
    assert kernels(lik.KERNEL_AUTO, full) == [cached]
    assert kernels(lik.KERNEL_AUTO, empty, full) == [generic, cached]
    assert kernels(lik.KERNEL_GENERIC, full) == [generic]
    assert kernels(lik.KERNEL_AUTO, full, empty) == [cached, cached]   # loaded by then
    assert not list(empty.iterdir())


SPECIES, SATURATING = 0, 1


def _chain(U, per, kinds):
    """U species in a chain, `per` terms out of each."""
    terms = [{"to": 0}]
    for s in range(U):
        for q in range(per):
            to = {"to": s + 1 + q} if s + 1 < U and s + 1 + q < U else {}
            terms.append(dict(frm=s, factors=[(kinds[(s + q) % len(kinds)], s, 3)], **to))
    return U, terms


def _hub(U, n):
    """n terms out of and into one species."""
    return U, [dict(frm=0, factors=[(SATURATING if k % 3 == 0 else SPECIES, k % U, 3)])
               for k in range(n)]


def _group_pairs(U, terms, cus=256):
    import ctypes
    arr = (lik.OdeTerm * len(terms))()
    for T, t in zip(arr, terms):
        T.frm, T.to, T.rate_param = t.get("frm", -1), t.get("to", -1), -1
        T.n_factors = len(t.get("factors", []))
        for j, factor in enumerate(t.get("factors", [])):
            T.kind[j], T.species[j], T.param[j] = factor
    m = lik.OdeModelC(U, 4, len(terms), ctypes.addressof(arr), None, 0, 0, 0, -1, 1.0,
                      (ctypes.c_int32 * 5)())
    f = getattr(lik.lib(), "_ZN3lik15ode_group_pairsERK13lik_ode_modelj")   # lik::ode_group_pairs
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_void_p, ctypes.c_uint32]
    return f(ctypes.byref(m), cus)


def test_deterministic_models_take_the_form_that_measured_faster():
    """Pairs up to which a group of lanes integrates one: none where the one-lane
    form was faster at 1,000 pairs already, and between the sizes that were
    measured on either side of the crossing elsewhere."""
    from paper_1606_08281_amd import workloads as W
    never = [_chain(1, 1, [SPECIES]), _chain(1, 1, [SATURATING]), _chain(2, 1, [SPECIES]),
             _chain(2, 3, [SATURATING, SPECIES]), _chain(4, 1, [SPECIES]),
             _chain(4, 15, [SATURATING, SPECIES]), _hub(8, 60), _hub(32, 100)]
    for U, terms in never:
        assert _group_pairs(U, terms) == 0, (U, len(terms))
    for (U, terms), above, below in [(_chain(8, 1, [SPECIES]), 4000, 16000),
                                     (_chain(8, 1, [SATURATING]), 32000, 49153),
                                     (_chain(16, 1, [SPECIES]), 16000, 32000),
                                     (_chain(17, 1, [SPECIES]), 16000, 32000),
                                     (_chain(32, 1, [SATURATING]), 49000, 49153)]:
        assert above <= _group_pairs(U, terms) < below, (U, len(terms))
    erk = W.erk_model()
    assert _group_pairs(erk["U"], erk["terms"]) == 49152
    assert _group_pairs(erk["U"], erk["terms"], cus=128) == 24576
    assert _group_pairs(8, _chain(8, 9, [SPECIES])[1][:65]) == 0     # more than four rounds of 16
