"""GPU: the one-cell-per-wave forms of mechanisms beside the named configurations:
third-body and falloff reactions on 16 lanes, unit counts at and just past the
rounds of the lane-group plan, gather plans of other rows, both layouts; bitwise
the lane-group kernels, whose 16-lane falloff form is checked against the oracle.
Every comparison first makes sure which kernels the two sides ran."""
import math
import os

import numpy as np
import pytest

from oracle import oracle as O
from paper_1309_2710_amd import synth
from tests import parity as PT

pytestmark = pytest.mark.gpu

THREADS = min(16, os.cpu_count() or 1)


@pytest.fixture(scope="module")
def R():
    from paper_1309_2710_amd import rkc
    rkc.lib()
    return rkc


def _pdep(cfg, seed):
    c = synth.CONFIGS[cfg]
    return synth.add_pressure_dependence(synth.config_mechanism(cfg), seed, 0.2, 0.2,
                                         T_ref=math.sqrt(c["T_range"][0] * c["T_range"][1]),
                                         P_ref=c["P_max"])


def _first_pairs(m, pairs):
    m = dict(m, n_reactions=2 * pairs)
    for k in ("reac", "prod", "A", "beta", "Ea", "pdep", "eff", "A0", "beta0", "Ea0", "troe"):
        m[k] = np.ascontiguousarray(m[k][:2 * pairs])
    return m


def _mech(name):
    """A named configuration, <cfg>+pd with pressure-dependent pairs, <cfg>/n with its
    first n pairs, or a set of the served workload (species, index)."""
    if isinstance(name, tuple):
        return synth.c5_mechanism(*name), "c2" if name[0] == 13 else "c3"
    cfg = name[:2] + ("p" if name[2:3] == "p" else "")
    m = _pdep(cfg, 1200 + int(cfg[1])) if "+pd" in name else synth.config_mechanism(cfg)
    return (_first_pairs(m, int(name.split("/")[1])) if "/" in name else m), cfg


def _run(R, gm, st, dt, layout=0, **kw):
    T, Y = st["T"].copy(), st["Y"].copy()
    if layout:
        Y = np.ascontiguousarray(Y.T)
    out = R.integrate(gm, T, st["P"], Y, dt, 1e-6, 1e-10, counters=True, stats=True,
                      layout=layout, **kw)
    return T, (Y.T if layout else Y), out


def _same(a, b):
    for x, y in ((a[0], b[0]), (a[1], b[1]), (a[2]["counters"], b[2]["counters"]),
                 (a[2]["status"], b[2]["status"])):
        assert np.array_equal(x, y)
    for k in ("n_rhs", "n_steps", "n_reject", "n_sigma", "n_power_iter", "s_max_used", "n_failed"):
        assert a[2]["stats"][k] == b[2]["stats"][k], k


# n: few cells, and (16 lanes) one more than the 3,072 that are resident
@pytest.mark.parametrize("name,n", [
    ("c2+pd", 300), ("c2+pd", 3073), ("c1+pd", 65), ("c2+pd/15", 33), ("c2+pd/16", 33),
    ("c2+pd/17", 33), ("c3p", 40), ("c3p/256", 33), ("c3p/257", 33), ("c4p", 20),
    ("c4p/768", 17), ("c4p/769", 17), ((13, 0), 300), ((53, 0), 300), ((53, 1), 1200),
    ("c3", 200), ("c4", 40)])
@pytest.mark.parametrize("method,layout", [(0, 0), (1, 1)])
def test_forms_equal_lane_groups(R, name, n, method, layout):
    print("[case] wave form", name, n, method, layout, flush=True)
    m, cfg = _mech(name)
    gm = R.Mechanism(m)
    st = synth.config_states(cfg, n, seed=300 + n)
    dt = 1e-7 if method == 0 and cfg in ("c1", "c2") else 1e-8
    a = _run(R, gm, st, dt, layout, method=method)
    b = _run(R, gm, st, dt, layout, method=method, schedule=R.SCHED_PLAIN)
    sa, sb = a[2]["stats"], b[2]["stats"]
    # 768 units are 12 rounds of 64 lanes: their table has no rounds for 4 x 4 waves
    has_form = name != "c4p/768"
    assert (sa["lds_bytes"] != sb["lds_bytes"]) == has_form, "not the kernels that were expected"
    _same(a, b)
    assert (a[2]["status"] == 0).all()


# the options and counts whose comparison elsewhere holds on either kernel: they do run
# the wave form (more cells than are resident, the recurrences of the coefficients, a
# capped stage count, few steps), but with a zero tolerance
@pytest.mark.parametrize("name,n,kw,wave", [
    ("c1", 3079, {}, True), ("c2", 3077, {}, True), ("c3", 2051, dict(method=1), True),
    ("c1", 33, dict(stage_coefs=1), True), ("c1", 33, dict(s_max=3), True),
    ("c1", 33, dict(max_steps=7), True), ("c1", 33, dict(layout=1), True),
    ("c1", 33, dict(lanes_per_cell=16), True), ("c1", 33, dict(lanes_per_cell=32), False),
    ("c1", 33, dict(block_groups=4), False), ("c1", 33, dict(atol=0.0), False)])
def test_which_calls_run_the_wave_form(R, name, n, kw, wave):
    print("[case] form of", name, n, kw, flush=True)
    m, cfg = _mech(name)
    gm = R.Mechanism(m)
    st = synth.config_states(cfg, n, seed=12)
    kw = dict(kw)
    atol, layout = kw.pop("atol", 1e-10), kw.get("layout", 0)
    res = []
    for more in ({}, dict(schedule=R.SCHED_PLAIN)):
        T, Y = st["T"].copy(), np.array(st["Y"].T if layout else st["Y"], order="C")
        out = R.integrate(gm, T, st["P"], Y, 1e-8, 1e-6, atol, counters=True, stats=True, **kw, **more)
        res.append((T, Y, out))
    a, b = res
    assert (a[2]["stats"]["lds_bytes"] != b[2]["stats"]["lds_bytes"]) == wave
    _same(a, b)


def test_small_falloff_set_against_oracle(R):
    print("[case] 16-lane falloff against the oracle", flush=True)
    m, cfg = _mech("c2+pd")
    c = synth.CONFIGS[cfg]
    st = synth.config_states(cfg, 400, seed=93)
    To, Yo, co = O.Model(m).integrate(st["T"], st["P"], st["Y"], c["dt"], c["rtol"], c["atol"],
                                      threads=THREADS)
    for kw in ({}, dict(schedule=R.SCHED_PLAIN)):
        T, Y, out = _run(R, R.Mechanism(m), st, c["dt"], **kw)
        assert (out["status"] == 0).all()
        PT.check(T, Y, out["counters"], To, Yo, co, c["rtol"], c["atol"], PT.max_flips("c2", 400))


# more cells than the wave form takes: the 16-lane groups hand their last ones over
@pytest.mark.parametrize("name,n,method,layout", [
    ("c2+pd", 13001, 0, 0), ("c2+pd", 62001, 1, 1), ("c1+pd", 13001, 0, 1), ("c1+pd", 62001, 1, 1),
    ((13, 0), 13001, 0, 0)])
def test_handed_over_cells_equal_plain(R, name, n, method, layout):
    print("[case] hand-over", name, n, method, layout, flush=True)
    m, cfg = _mech(name)
    gm = R.Mechanism(m)
    st = synth.config_states(cfg, n, seed=n)
    dt = 1e-7 if method == 0 else 1e-8
    a = _run(R, gm, st, dt, layout, method=method)
    b = _run(R, gm, st, dt, layout, method=method, schedule=R.SCHED_PLAIN)
    _same(a, b)
    assert a[2]["stats"]["n_rhs"] <= a[2]["stats"]["n_rhs_slots"]
    # cells of 6 evaluations each (13 species, RKCK) end before any could be handed over
    if (name, method) != ("c2+pd", 1):
        assert a[2]["stats"]["n_rhs_slots"] < b[2]["stats"]["n_rhs_slots"]


def test_graph_with_hand_over_equals_eager(R):
    """A recorded step whose 16-lane groups hand over, replayed with eager hand-overs
    of the same handle and other sizes between."""
    import torch
    print("[case] graph with hand-over", flush=True)
    n, dt = 13000, 1e-7
    gm = R.Mechanism(synth.config_mechanism("c1"))
    st = synth.config_states("c1", n, seed=8)
    T0, P, Y0 = (torch.from_numpy(st[k]).cuda() for k in ("T", "P", "Y"))
    Te, Ye = T0.clone(), Y0.clone()
    R.integrate(gm, Te, P, Ye, dt, 1e-6, 1e-10, status=False)
    T, Y = T0.clone(), Y0.clone()
    g = R.Graph(gm, T, P, Y, dt, 1e-6, 1e-10)
    for k in range(4):
        T.copy_(T0)
        Y.copy_(Y0)
        g.launch()
        torch.cuda.synchronize()
        assert torch.equal(T, Te) and torch.equal(Y, Ye), k
        r = torch.arange(n + 3000 * (k + 1), device="cuda") % n
        Tb, Yb = T0[r].contiguous(), Y0[r].contiguous()
        R.integrate(gm, Tb, P[r].contiguous(), Yb, dt, 1e-6, 1e-10, status=False)
        assert torch.equal(Tb, Te[r]) and torch.equal(Yb, Ye[r]), k
    g.close()
