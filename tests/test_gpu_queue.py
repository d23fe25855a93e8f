"""GPU: a queued launch gives every cell the bits of the plain schedule, whatever
the resident grid (so however the queue's parts run out), the cost order of its
cells, bad input among them, and the caller's capture (index order)."""
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


def _run(R, gm, st, dt, method, **kw):
    T, Y = st["T"].copy(), st["Y"].copy()
    out = R.integrate(gm, T, st["P"], Y, dt, 1e-6, 1e-10, method=method, counters=True, **kw)
    return T, Y, out["counters"], out["status"], out.get("stats")


# grids of 1, 3 and 17 workgroups of 1 or 3 lane groups: fewer cells than groups,
# one more, parts of unequal length, and past the 4,096 cells one workgroup sorts
@pytest.mark.parametrize("cfg,G,method,grid,groups,n", [
    ("c1", 16, 0, 1, 3, 2), ("c1", 16, 0, 1, 3, 4), ("c1", 16, 0, 17, 3, 52), ("c1", 16, 1, 3, 1, 19),
    ("c1", 16, 1, 17, 3, 4097), ("c2", 32, 1, 17, 1, 8193), ("c3", 64, 0, 17, 1, 50),
    ("c3p", 64, 1, 3, 3, 41), ("c4", 64, 1, 3, 1, 20), ("ab", 8, 0, 3, 3, 301), ("ab", 8, 1, 1, 1, 33)])
def test_queue_equals_plain(R, cfg, G, method, grid, groups, n):
    print("[case] queue", cfg, G, method, grid, groups, n, flush=True)
    if cfg == "ab":
        m = mechs.a_to_b(k=3e7)
        a = np.linspace(0.1, 0.9, n)
        st = {"T": np.full(n, 1000.0), "P": np.full(n, 101325.0), "Y": np.stack([a, 1.0 - a], 1)}
    else:
        m = synth.config_mechanism(cfg)
        st = synth.config_states(cfg, n, seed=40 + n)
    if n > 3:
        st["T"][0], st["P"][1], st["Y"][n - 1, 0] = np.nan, -1.0, np.inf
        st["T"][2] = 20.0   # rates overflow: an infinite cost
    gm = R.Mechanism(m)
    dt = 1e-8 if cfg != "ab" else 1e-6
    a = _run(R, gm, st, dt, method, lanes_per_cell=G, schedule=R.SCHED_PERSISTENT, grid_blocks=grid,
             block_groups=groups)
    b = _run(R, gm, st, dt, method, lanes_per_cell=G, schedule=R.SCHED_PLAIN, block_groups=groups)
    for x, y in zip(a[:4], b[:4]):
        assert np.array_equal(x, y, equal_nan=x.dtype == np.float64)
    if n > 3:
        assert (a[3][[0, 1, n - 1]] == 4).all()


@pytest.mark.parametrize("cfg,method", [("c1", 1), ("c3", 0)])
def test_captured_call_and_graph_equal_eager(R, cfg, method):
    """More cells than are resident: an ordered graph, and a capture by the
    caller, each replayed with eager ordered calls of other sizes between."""
    import torch
    n = {"c1": 20000, "c3": 5000}[cfg]
    gm = R.Mechanism(synth.config_mechanism(cfg))
    st = synth.config_states(cfg, n, seed=3)
    T0, P, Y0 = (torch.from_numpy(st[k]).cuda() for k in ("T", "P", "Y"))
    dt = 1e-8
    Te, Ye = T0.clone(), Y0.clone()
    R.integrate(gm, Te, P, Ye, dt, 1e-6, 1e-10, method=method, status=False)
    T, Y = T0.clone(), Y0.clone()
    graph = R.Graph(gm, T, P, Y, dt, 1e-6, 1e-10, method=method)
    torch.cuda.synchronize()
    cap = torch.cuda.CUDAGraph()
    Tc, Yc = T0.clone(), Y0.clone()
    with torch.cuda.graph(cap):
        R.integrate(gm, Tc, P, Yc, dt, 1e-6, 1e-10, method=method, status=False)
    for k in range(3):
        for x, x0 in ((T, T0), (Y, Y0), (Tc, T0), (Yc, Y0)):
            x.copy_(x0)
        graph.launch()
        cap.replay()
        torch.cuda.synchronize()
        assert torch.equal(T, Te) and torch.equal(Y, Ye), k
        assert torch.equal(Tc, Te) and torch.equal(Yc, Ye), k
        r = torch.arange(n + 5000 * (k + 1), device="cuda") % n
        Tb, Yb = T0[r].contiguous(), Y0[r].contiguous()
        R.integrate(gm, Tb, P[r].contiguous(), Yb, dt, 1e-6, 1e-10, method=method, status=False)
        assert torch.equal(Tb, Te[r]) and torch.equal(Yb, Ye[r]), k
    graph.close()


# 16-lane groups hand the cells they have left to one wave each: when every cell
# was resident, when they queued, both methods, and steps whose stage counts or
# error estimates take the rare branches
@pytest.mark.parametrize("cfg,n,method,dt,kw", [
    ("c1", 13000, 0, 1e-7, {}), ("c1", 62001, 1, 1e-8, {}), ("c2", 20001, 0, 1e-6, {}),
    ("c2", 13001, 0, 1e-7, dict(stage_coefs=1)), ("c1", 13001, 0, 1e-6, dict(max_steps=40)),
    ("c1", 13003, 0, 3e-7, dict(s_max=3)), ("c2", 13003, 0, 1e-6, dict(layout=1))])
def test_handed_over_cells_equal_plain(R, cfg, n, method, dt, kw):
    print("[case] hand-over", cfg, n, method, kw, flush=True)
    st = synth.config_states(cfg, n, seed=n)
    if kw.get("layout"):
        st["Y"] = np.ascontiguousarray(st["Y"].T)
    gm = R.Mechanism(synth.config_mechanism(cfg))
    a = _run(R, gm, st, dt, method, stats=True, **kw)
    b = _run(R, gm, st, dt, method, stats=True, schedule=R.SCHED_PLAIN, **kw)
    for x, y in zip(a[:4], b[:4]):
        assert np.array_equal(x, y)
    for k in ("n_rhs", "n_steps", "n_reject", "n_sigma", "n_power_iter", "s_max_used", "n_failed"):
        assert a[4][k] == b[4][k], k
    assert a[4]["n_rhs"] <= a[4]["n_rhs_slots"] < b[4]["n_rhs_slots"]
