"""GPU: the one-cell-per-wave kernels give bitwise the lane-group kernels' results
(state, status and counters), so the automatic choice between them by cell
count never changes a cell.  The sizes sit at the edges of the launch: one
cell, one cell per compute unit and one more, more cells than are resident.
The stage counts past the coefficient table (recurrences), tiny tolerances
and bad input are the remaining branches."""
import numpy as np
import pytest

from paper_1309_2710_amd import synth
from tests import mechs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    from paper_1309_2710_amd import rkc
    rkc.lib()
    return rkc


def _both(R, m, st, dt, rtol, atol, **kw):
    """(T, Y, out) of the automatic launch and of the lane-group kernels."""
    gm = R.Mechanism(m)
    res = []
    for sched in (R.SCHED_AUTO, R.SCHED_PLAIN):
        T, Y = st["T"].copy(), st["Y"].copy()
        out = R.integrate(gm, T, st["P"], Y, dt, rtol, atol, counters=True, stats=True,
                          schedule=sched, **kw)
        res.append((T, Y, out))
    return res


def _same(a, b):
    assert np.array_equal(a[0], b[0], equal_nan=True) and np.array_equal(a[1], b[1], equal_nan=True)
    assert np.array_equal(a[2]["counters"], b[2]["counters"])
    assert np.array_equal(a[2]["status"], b[2]["status"])
    for k in ("n_rhs", "n_steps", "n_reject", "n_sigma", "n_power_iter", "s_max_used", "n_failed"):
        assert a[2]["stats"][k] == b[2]["stats"][k], k


# the resident cells of the forms: 16-lane sets 12 per compute unit, 53 species 4
# (two waves a cell) then 8, with falloff 8, 111 species 1 (8 waves a cell) then 2
@pytest.mark.parametrize("cfg,n,method", [
    ("c1", 1, 0), ("c1", 257, 0), ("c1", 3079, 0), ("c1", 130, 1), ("c2", 3077, 0), ("c2", 515, 1),
    ("c3", 1, 0), ("c3", 259, 0), ("c3", 1153, 0), ("c3", 2051, 1), ("c3p", 3, 0), ("c3p", 513, 1),
    ("c4", 2, 0), ("c4", 256, 1), ("c4", 261, 0), ("c4p", 5, 0), ("c4p", 260, 1)])
def test_wave_equals_lane_groups(R, cfg, n, method):
    print("[case] wave", cfg, n, method, flush=True)
    dt = 1e-8 if method == 1 or cfg in ("c4", "c4p") else 1e-7
    st = synth.config_states(cfg, n, seed=900 + n)
    a, b = _both(R, synth.config_mechanism(cfg), st, dt, 1e-6, 1e-10, method=method)
    assert a[2]["stats"]["block_threads"] != b[2]["stats"]["block_threads"] or n > 2000
    _same(a, b)
    assert (a[2]["status"] == 0).all()


@pytest.mark.parametrize("kw", [dict(stage_coefs=1), dict(s_max=3), dict(max_steps=7),
                                dict(layout=1)])
def test_wave_options(R, kw):
    print("[case] wave options", kw, flush=True)
    st = synth.config_states("c1", 33, seed=71)
    if kw.get("layout"):
        st["Y"] = np.ascontiguousarray(st["Y"].T)
    _same(*_both(R, synth.config_mechanism("c1"), st, 1e-7, 1e-6, 1e-10, **kw))


def test_wave_stage_count_past_the_table(R):
    """A -> B with k dt = 3e4 needs up to 176 stages, past the 128 tabulated ones."""
    m = mechs.a_to_b(k=3e10)
    n = 5
    st = {"T": np.full(n, 1000.0), "P": np.full(n, 101325.0),
          "Y": np.stack([np.linspace(0.1, 0.9, n), 1.0 - np.linspace(0.1, 0.9, n)], 1)}
    a, b = _both(R, m, st, 1e-6, 1e-6, 1e-10)
    assert a[2]["stats"]["s_max_used"] > 128
    _same(a, b)


@pytest.mark.parametrize("cfg,n", [("c1", 40), ("c3", 40), ("c4", 9)])
def test_wave_bad_input_and_zero_tolerance(R, cfg, n):
    print("[case] wave bad input", cfg, flush=True)
    st = synth.config_states(cfg, n, seed=5)
    st["T"][1] = -3.0
    st["T"][4] = np.nan
    st["P"][2] = 0.0
    st["Y"][5, 3] = np.inf
    st["T"][6] = 20.0       # rates overflow
    m = synth.config_mechanism(cfg)
    a, b = _both(R, m, st, 1e-8, 1e-6, 1e-10)
    assert set(a[2]["status"][[1, 2, 4, 5]]) == {4}
    _same(a, b)
    _same(*_both(R, m, st, 1e-9, 1e-6, 0.0))   # atol 0: lane groups on both sides
