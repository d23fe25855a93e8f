"""GPU: a recorded step keeps queue scratch only where its cells queue (6 bytes a
cell) and hand-over records only where its lane groups hand over (1.5 MB): eight
recorded steps of each kind against the device's free memory."""
import pytest

from paper_1309_2710_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    from paper_1309_2710_amd import rkc
    rkc.lib()
    return rkc


# all cells in the plain schedule (12.6 MB of scratch per step before), one lane per
# cell, few cells in the wave form (1.5 MB of records before), and queues of more
# rounds of cells than are ordered (6.3 MB)
@pytest.mark.parametrize("n,kw", [
    (1 << 21, dict(schedule=1)), (1 << 21, dict(lanes_per_cell=1)), (64, {}),
    (1 << 20, dict(lanes_per_cell=32, grid_blocks=1)),
    (1 << 20, dict(lanes_per_cell=32, grid_blocks=1, method=1))])
def test_scratch_only_where_used(R, n, kw):
    import torch
    print("[case] graph memory", n, kw, flush=True)
    gm = R.Mechanism(synth.config_mechanism("c1"))
    T = torch.full((n,), 1200.0, dtype=torch.float64, device="cuda")
    P = torch.full((n,), 101325.0, dtype=torch.float64, device="cuda")
    Y = torch.full((n, 9), 1.0 / 9.0, dtype=torch.float64, device="cuda")
    keep = [R.Graph(gm, T, P, Y, 1e-8, **kw)]   # tables and the runtime's own first use
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    keep += [R.Graph(gm, T, P, Y, 1e-8, **kw) for _ in range(8)]
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    print("used", used, flush=True)
    for g in keep:
        g.close()
    # counters and queue heads: 3.2 KB a step, in pages of 2 MB
    assert used <= 4 << 20
