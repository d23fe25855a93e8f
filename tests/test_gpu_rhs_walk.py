"""GPU: a source-term launch whose grid walks over the cells gives every cell the
bits it has as the only turn of its lane group."""
import pytest

from paper_1309_2710_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    from paper_1309_2710_amd import rkc
    rkc.lib()
    return rkc


# the source term's grid walks over the cells: one cell, part of a workgroup, one
# more than a chip's worth of lane groups (16,384 of 16 lanes, 4,096 of 64, fewer
# resident for the falloff and 111-species sets), and a few turns
@pytest.mark.parametrize("cfg,n", [
    ("c1", 1), ("c1", 16385), ("c2", 33333), ("c3", 5), ("c3", 4097), ("c3p", 8193), ("c4", 3),
    ("c4", 2500), ("c4p", 1031)])
@pytest.mark.parametrize("layout", [0, 1])
def test_rhs_walk_equals_single_turns(R, cfg, n, layout):
    import torch
    print("[case] rhs walk", cfg, n, layout, flush=True)
    gm = R.Mechanism(synth.config_mechanism(cfg))
    st = synth.config_states(cfg, n, seed=6)
    T, P, Y = (torch.from_numpy(st[k]).cuda() for k in ("T", "P", "Y"))
    f = R.rhs(gm, T, P, Y.t().contiguous() if layout else Y, layout=layout)
    f = f.t() if layout else f
    for a in range(0, n, 128):
        s = slice(a, a + 128)
        one = R.rhs(gm, T[s].contiguous(), P[s].contiguous(), Y[s].contiguous())
        assert torch.equal(f[s], one), a
