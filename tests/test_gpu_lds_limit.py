"""GPU: a mechanism whose tables nearly fill LDS.  Queued launches of it have no room
for the counts of the cost classes beside the tables and take their cells in index
order; recorded steps likewise.  Results are those of the plain schedule."""
import numpy as np
import pytest

from tests import mechs

pytestmark = pytest.mark.gpu

LDS = 160 * 1024
N_SPECIES = 50


@pytest.fixture(scope="module")
def R():
    from paper_1309_2710_amd import rkc
    rkc.lib()
    return rkc


def _mech(rounds):
    """64 slow first-order reactions of 50 species per round of 64 lanes."""
    rx = []
    for j in range(64 * rounds):
        a, b = j % N_SPECIES, (j + 1 + j // N_SPECIES) % N_SPECIES
        rx.append(([a], [b if b != a else (a + 1) % N_SPECIES], 1e3 * (1 + j % 7), 0.0, 0.0))
    return mechs.tiny([10.0 + i for i in range(N_SPECIES)], rx)


def _states(n):
    rng = np.random.default_rng(4)
    return {"T": rng.uniform(900.0, 1500.0, n), "P": np.full(n, 101325.0),
            "Y": rng.dirichlet(np.ones(N_SPECIES), size=n)}


def _run(R, gm, st, **kw):
    T, Y = st["T"].copy(), st["Y"].copy()
    out = R.integrate(gm, T, st["P"], Y, 1e-5, 1e-6, 1e-10, counters=True, stats=True, check=False,
                      **kw)
    return T, Y, out


@pytest.fixture(scope="module")
def largest(R):
    """The largest of these mechanisms that a plain launch takes."""
    gm = None
    for rounds in range(24, 40):
        m = R.Mechanism(_mech(rounds))
        if _run(R, m, _states(4), schedule=R.SCHED_PLAIN)[2]["rc"] != R.OK:
            break
        gm = m
    return gm


@pytest.mark.parametrize("method", [0, 1])
def test_queued_launch_without_room_for_classes(R, largest, method):
    print("[case] LDS limit, method", method, flush=True)
    st = _states(700)
    b = _run(R, largest, st, method=method, schedule=R.SCHED_PLAIN)
    assert b[2]["rc"] == R.OK and LDS - 8192 < b[2]["stats"]["lds_bytes"] <= LDS
    a = _run(R, largest, st, method=method)
    assert a[2]["rc"] == R.OK and a[2]["stats"]["schedule"] == R.SCHED_PERSISTENT
    assert a[2]["stats"]["grid_blocks"] * a[2]["stats"]["block_threads"] // 64 < 700
    for x, y in ((a[0], b[0]), (a[1], b[1]), (a[2]["counters"], b[2]["counters"])):
        assert np.array_equal(x, y)


# every cell resident, and cells that queue
@pytest.mark.parametrize("n", [40, 700])
def test_recorded_step_without_room_for_classes(R, largest, n):
    import torch
    print("[case] LDS limit, graph", n, flush=True)
    st = _states(n)
    Te, Ye, _ = _run(R, largest, st, schedule=R.SCHED_PLAIN)
    T, P, Y = (torch.from_numpy(st[k].copy()).cuda() for k in ("T", "P", "Y"))
    T0, Y0 = T.clone(), Y.clone()
    g = R.Graph(largest, T, P, Y, 1e-5, 1e-6, 1e-10)
    for _ in range(3):
        T.copy_(T0)
        Y.copy_(Y0)
        g.launch()
        torch.cuda.synchronize()
        assert np.array_equal(T.cpu().numpy(), Te) and np.array_equal(Y.cpu().numpy(), Ye)
    g.close()
