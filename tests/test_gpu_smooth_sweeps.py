"""The smoothed TNS's sweeps as resident grids against one launch per level:
the same operations in the same order, so equal bit for bit, under every net
model and precision, on designs with more and fewer chunks than waves, with
several backward passes after one forward, and again after changed positions.
Values against the oracle are tested elsewhere."""
import numpy as np
import pytest
import torch

from paper_2503_11674_amd import netgen
from tests.conftest import with_clock

pytestmark = pytest.mark.gpu


def _design(library, cells, depth, fanout_cap=12, fanin_hi=4):
    cfg = netgen.NetlistConfig("s", cells, ff_frac=0.15, depth=depth, fanin_lo=1, fanin_hi=fanin_hi,
                               fanout_cap=fanout_cap, die=15.0 * cells ** 0.5, seed=2)
    return with_clock(netgen.make_netlist(cfg), library, 0.3)


def _xy(nl, seed):
    return [torch.tensor(a, device="cuda") for a in netgen.jitter_positions(nl, 20.0, seed)]


def _passes(g, nl, mode):
    if mode is not None:
        g.set_tuning(sweep_mode=mode)
    out = []
    g.sta_update(*_xy(nl, 1))
    one = torch.ones((), dtype=torch.float64, device="cuda")
    for seed, gamma in ((1, 10.0), (2, 3.0), (3, 40.0)):
        v = g.stns_fwd(*_xy(nl, seed), gamma)
        out.append(float(v))
        for _ in range(2):
            gx = torch.zeros(nl["num_cells"], device="cuda")
            gy = torch.zeros_like(gx)
            g.stns_bwd(one, gx, gy)
            out += [gx.cpu().numpy(), gy.cpu().numpy()]
    return out


@pytest.mark.parametrize("cells,depth,prec,model,fanin_hi", [
    (60, 3, "f32", 0, 4), (700, 9, "f32", 0, 20), (5000, 40, "f32", 1, 4), (3000, 12, "f32", 2, 4),
    (700, 9, "f64", 0, 4), (2000, 7, "f64", 2, 40), (150_000, 12, "f32", 0, 4)])
def test_grids_and_levels_agree(library, cells, depth, prec, model, fanin_hi):
    from paper_2503_11674_amd import tdp
    nl = _design(library, cells, depth, fanin_hi=fanin_hi, fanout_cap=60 if fanin_hi > 20 else 12)
    res = []
    for mode in (0, None):
        g = tdp.TimingGraph(nl, dict(library, net_model=model), precision=prec, max_paths=10, max_k=1)
        res.append(_passes(g, nl, mode))
        g.close()
    assert np.abs(res[0][1]).max() > 0
    for a, b in zip(*res):
        assert np.array_equal(a, b)


def test_a_net_wider_than_a_chunk(library):
    """Forward as a grid, backward by levels."""
    from paper_2503_11674_amd import tdp
    nl = _design(library, 900, 6)
    nl = dict(nl, net_ptr=nl["net_ptr"].copy(), net_pins=nl["net_pins"].copy())
    ptr, pins = nl["net_ptr"], nl["net_pins"]
    drv = pins[ptr[:-1]]
    sinks = [list(pins[a + 1:b]) for a, b in zip(ptr[:-1], ptr[1:])]
    ports = np.nonzero(nl["pin_cell"][drv] < 0)[0]
    for n in ports[1:]:
        if len(sinks[ports[0]]) < 90:
            sinks[ports[0]] += sinks[n]
            sinks[n] = []
    assert len(sinks[ports[0]]) > 63
    ptr[1:] = np.cumsum([1 + len(s) for s in sinks])
    nl["net_pins"] = np.concatenate([[d] + s for d, s in zip(drv, sinks)]).astype(np.int32)
    res = []
    for mode in (0, None):
        g = tdp.TimingGraph(nl, library, max_paths=10, max_k=1)
        res.append(_passes(g, nl, mode))
        g.close()
    for a, b in zip(*res):
        assert np.array_equal(a, b)


def test_positions_that_are_not_finite_end(library):
    """NaN of every payload passes through the published words."""
    from paper_2503_11674_amd import tdp
    nl = _design(library, 700, 9)
    g = tdp.TimingGraph(nl, library, max_paths=10, max_k=1)
    x, y = _xy(nl, 1)
    g.sta_update(x, y)
    want = float(g.stns_fwd(x, y, 10.0))
    bad = x.view(torch.int32).clone()
    bad[::3] = -1
    bad[1::3] = 0x7f800000
    assert not np.isfinite(float(g.stns_fwd(bad.view(torch.float32), y, 10.0)))
    gx = torch.zeros(nl["num_cells"], device="cuda")
    g.stns_bwd(torch.ones((), dtype=torch.float64, device="cuda"), gx, torch.zeros_like(gx))
    torch.cuda.synchronize()
    assert float(g.stns_fwd(x, y, 10.0)) == want
    g.close()
