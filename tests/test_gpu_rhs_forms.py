"""GPU: the source term's launch forms give every cell the same bits: one turn of
512-lane workgroups (the most cells they reach, 512 lanes on each of 256 compute
units, and one more), one turn of the largest workgroups, and a grid that walks;
both layouts."""
import pytest

from paper_1309_2710_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    from paper_1309_2710_amd import rkc
    rkc.lib()
    return rkc


# 16 lanes: 8,192 cells at once in 512-lane workgroups, 16,384 in 1,024; 64 lanes 2,048
# and 4,096; falloff in 32 lanes and two slots 4,096 and 6,144; 111 species 2,048 and
# 3,072 (fewer with falloff, where LDS ends at ten groups)
@pytest.mark.parametrize("cfg,sizes", [
    ("c1", (8192, 8193, 16384, 16385)), ("c3", (2048, 2049, 4096, 4097)),
    ("c3p", (4096, 4097, 6144, 6145)), ("c4", (2048, 2049, 3072, 3073)),
    ("c4p", (2048, 2049, 2817, 3073))])
@pytest.mark.parametrize("layout", [0, 1])
def test_rhs_forms_agree(R, cfg, sizes, layout):
    import torch
    gm = R.Mechanism(synth.config_mechanism(cfg))
    n = max(sizes)
    st = synth.config_states(cfg, n, seed=16)
    T, P, Y = (torch.from_numpy(st[k]).cuda() for k in ("T", "P", "Y"))
    one = torch.cat([R.rhs(gm, T[a:a + 100].contiguous(), P[a:a + 100].contiguous(),
                           Y[a:a + 100].contiguous()) for a in range(0, n, 100)])
    for k in sizes:
        print("[case] rhs forms", cfg, k, layout, flush=True)
        y = Y[:k].t().contiguous() if layout else Y[:k].contiguous()
        f = R.rhs(gm, T[:k].contiguous(), P[:k].contiguous(), y, layout=layout)
        assert torch.equal(f.t() if layout else f, one[:k]), k
