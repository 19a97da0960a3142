"""The backward sweep of designs large enough for the drivers to publish their
cells' inputs: required times and slacks bit for bit those of one launch per
level, in updates of one call and of two, with cells of more inputs than are
loaded ahead, in both precisions."""
import numpy as np
import pytest
import torch

from paper_2503_11674_amd import netgen
from tests.conftest import with_clock

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,fanin_hi", [("f32", 4), ("f32", 11), ("f64", 4)])
def test_drivers_publish_their_inputs(library, prec, fanin_hi):
    from paper_2503_11674_amd import tdp
    cells = 1_100_000 if fanin_hi == 4 else 700_000
    cfg = netgen.NetlistConfig("b", cells, ff_frac=0.12, depth=14, fanin_lo=2, fanin_hi=fanin_hi, fanout_cap=20,
                               die=8000.0, seed=6)
    nl = with_clock(netgen.make_netlist(cfg), library, 0.2)
    g = tdp.TimingGraph(nl, library, precision=prec, max_paths=10, max_k=1)
    # net chunks hold 64 pins, and 256 chunks a compute unit are the rule
    assert nl["num_pins"] / 64 > 256 * torch.cuda.get_device_properties(0).multi_processor_count
    xs = [[torch.tensor(a, device="cuda") for a in netgen.jitter_positions(nl, 30.0, s)] for s in (1, 2)]
    g.set_tuning(sweep_mode=0)
    want = []
    for x, y in xs:
        g.sta_update(x, y)
        want.append({k: v.cpu().numpy() for k, v in g.export().items()})
    g.close()
    g = tdp.TimingGraph(nl, library, precision=prec, max_paths=10, max_k=1)
    for i in (0, 1, 0):
        if i == 1:
            g.sta_update_arrivals(*xs[i])
            g.sta_update_required()
        else:
            g.sta_update(*xs[i])
        got = {k: v.cpu().numpy() for k, v in g.export().items()}
        for k in want[i]:
            assert np.array_equal(got[k], want[i][k]), k
    g.close()
