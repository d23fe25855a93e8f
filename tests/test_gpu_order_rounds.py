"""GPU: queues of exactly as many rounds of cells as are ordered (64 of RKC, 32 of
RKCK) and of one cell more give every cell the bits of the plain schedule."""
import numpy as np
import pytest

from paper_1309_2710_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    from paper_1309_2710_amd import rkc
    rkc.lib()
    return rkc


# 51 resident groups, and 1,088 whose cells take nine of the sort's workgroups
@pytest.mark.parametrize("cfg,G,method,grid,groups", [
    ("c1", 16, 0, 17, 3), ("c1", 16, 1, 17, 3), ("c1", 16, 1, 17, 64), ("c3p", 32, 1, 5, 3)])
@pytest.mark.parametrize("more", [0, 1])
def test_rounds_equal_plain(R, cfg, G, method, grid, groups, more):
    n = (32 if method else 64) * grid * groups + more
    print("[case] order rounds", cfg, G, method, n, flush=True)
    st = synth.config_states(cfg, n, seed=n)
    st["T"][n // 2] = -1.0
    gm = R.Mechanism(synth.config_mechanism(cfg))
    res = []
    for kw in (dict(schedule=R.SCHED_PERSISTENT, grid_blocks=grid), dict(schedule=R.SCHED_PLAIN)):
        T, Y = st["T"].copy(), st["Y"].copy()
        out = R.integrate(gm, T, st["P"], Y, 1e-8, 1e-6, 1e-10, method=method, lanes_per_cell=G,
                          block_groups=groups, counters=True, **kw)
        res.append((T, Y, out["counters"], out["status"]))
    for x, y in zip(*res):
        assert np.array_equal(x, y)
    assert res[0][3][n // 2] == R.CELL_BADINPUT and (np.delete(res[0][3], n // 2) == 0).all()
