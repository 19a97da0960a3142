"""Waits that run out of polls: the kernels end, every call that reads results
to the host reports it, and the next normal pass is right again.  The waits are
made to run out from the host, by start points that are never published or by a
budget of a few polls."""
import numpy as np
import pytest
import torch

from paper_2503_11674_amd import netgen
from tests.conftest import with_clock

pytestmark = pytest.mark.gpu

DEVICE_ERROR = 4


def _design(library, cells, depth, seed=5):
    cfg = netgen.NetlistConfig("g", cells, ff_frac=0.15, depth=depth, fanin_lo=1, fanin_hi=4, fanout_cap=12,
                               die=15.0 * cells ** 0.5, seed=seed)
    return with_clock(netgen.make_netlist(cfg), library, 0.3)


def _xy(*nls):
    return [torch.tensor(np.concatenate([nl[a] for nl in nls]), device="cuda") for a in ("x", "y")]


def _reports(tdp, call):
    with pytest.raises(tdp.TdpError) as e:
        call()
    assert e.value.status == DEVICE_ERROR


def test_batch_summary_reports_a_sweep_that_gave_up(library):
    from paper_2503_11674_amd import tdp
    nls = [_design(library, n, 12, seed=n) for n in (300, 700, 500)]
    g = tdp.TimingGraph(nls, library, max_paths=100, max_k=4)
    x, y = _xy(*nls)
    g.sta_update(x, y)
    want = g.batch_summary()
    g.set_tuning(spin_log2=4, sweep_mode=2)
    g.sta_update(x, y)
    _reports(tdp, g.batch_summary)
    _reports(tdp, g.summary)
    g.set_tuning(spin_log2=20, sweep_mode=1)
    g.sta_update(x, y)
    for a, b in zip(want, g.batch_summary()):
        assert np.array_equal(a, b)
    g.close()
