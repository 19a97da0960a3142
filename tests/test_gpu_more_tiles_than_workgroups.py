"""Designs so large that the one-launch prefix sums have more tiles than
workgroups (a workgroup then takes several): the violated endpoints beyond 512
tiles of 4,096, the pair list beyond 512 tiles of 16,384 sinks, the cells' lists
beyond 512 tiles of 4,096 cells.  Against the same selections and sums in numpy
from the slacks and paths that the library gives (pinned elsewhere at all
smaller sizes)."""
import numpy as np
import pytest
import torch

from paper_2503_11674_amd import netgen

pytestmark = pytest.mark.gpu

W0, W1 = 10.0, 0.2


def _pairs_and_loss(g, nl, x, y, p, wns):
    """P, its weights (Eq. 9 from an empty P), the pin-to-pin loss and gradient."""
    g.pairs_reset()
    assert g.pairs_count() == 0
    g.pairs_update(rule=0, w0=W0, w1=W1)
    w, in_p = g.pairs_export()
    ptr, pins = p["path_ptr"], p["path_pins"]
    share = p["path_slack"].astype(np.float64) / wns
    path = np.repeat(np.arange(p["num_paths"]), np.diff(ptr))
    sinks = (np.arange(len(pins)) - ptr[path]) % 2 == 1  # every second pin of a path
    pin, path = pins[sinks], path[sinks]
    total = np.zeros(nl["num_pins"])
    np.add.at(total, pin, share[path])
    first = np.full(nl["num_pins"], p["num_paths"])
    np.minimum.at(first, pin, path)
    member = first < p["num_paths"]
    assert np.array_equal(in_p.astype(bool), member) and g.pairs_count() == member.sum() > 0
    want = W0 + W1 * (total[member] - share[first[member]])
    assert np.abs(w[member] - want).max() <= 1e-5 * want.max() and not w[~member].any()
    drv = np.empty(nl["num_pins"], np.int64)
    size = np.diff(nl["net_ptr"])
    drv[nl["net_pins"]] = np.repeat(nl["net_pins"][nl["net_ptr"][:-1]], size)
    t = np.nonzero(member)[0]
    s = drv[t]

    def coord(pin, c, off):
        cell = nl["pin_cell"][pin]
        return np.where(cell >= 0, c[cell], 0.0).astype(np.float64) + off[pin]

    dx = coord(s, nl["x"], nl["pin_off_x"]) - coord(t, nl["x"], nl["pin_off_x"])
    dy = coord(s, nl["y"], nl["pin_off_y"]) - coord(t, nl["y"], nl["pin_off_y"])
    loss = float(g.p2p_loss_fwd(x, y))
    assert abs(loss - (w[t] * (dx * dx + dy * dy)).sum()) <= 1e-5 * loss
    gx, gy = torch.zeros_like(x), torch.zeros_like(y)
    g.p2p_loss_bwd(x, y, torch.ones((), dtype=torch.float64, device="cuda"), gx, gy)
    for got, d in ((gx, dx), (gy, dy)):
        ref = np.zeros(nl["num_cells"])
        for pin, sign in ((s, 2.0), (t, -2.0)):
            cell = nl["pin_cell"][pin]
            ok = cell >= 0
            np.add.at(ref, cell[ok], (sign * w[t] * d)[ok])
        ref[np.asarray(nl["cell_fixed"]) != 0] = 0.0
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("cells,ff,lo", [(2_340_000, 0.9, 1), (2_650_000, 0.05, 3)])
def test_more_tiles_than_workgroups(library, cells, ff, lo):
    from paper_2503_11674_amd import tdp
    cfg = netgen.NetlistConfig("big", cells, ff_frac=ff, depth=6, fanin_lo=lo, fanin_hi=4, fanout_cap=60 if ff > 0.5 else 16,
                               die=8.0 * cells ** 0.5, seed=2)
    nl = netgen.make_netlist(cfg)
    nl["clock_period"] = np.float32(1000.0)
    g = tdp.TimingGraph(nl, library, max_paths=max(1000, int(1.2 * cells * ff)), max_k=1)
    x, y = [torch.tensor(nl[a], device="cuda") for a in ("x", "y")]
    g.sta_update(x, y)
    ends = np.asarray(nl["cell_in_pins"])[np.asarray(nl["cell_in_ptr"])[:-1][np.asarray(nl["cell_is_ff"]) != 0]]
    at = g.export()["at"].cpu().numpy()[ends]
    g.set_clock(float(np.quantile(at, 0.3)))
    g.sta_update(x, y)
    slack = g.export()["slack"].cpu().numpy()[ends]
    wns, _, n_fail = g.summary()
    if ff > 0.5:
        assert len(ends) > 512 * 4096
    else:
        assert g.num_sinks > 512 * 16384
    assert nl["num_cells"] > 512 * 4096 and n_fail == (slack < 0).sum() > 1000
    for n in (-1, 70_000):
        g.extract_paths(n=n, k=1)
        p = g.paths()
        order = np.lexsort((ends, slack))
        take = order[: n_fail if n < 0 else n]
        assert np.array_equal(p["path_ep"], ends[take]) and np.array_equal(p["path_slack"], slack[take].astype(np.float32))
        keep = p["path_slack"] < 0
        if keep.all():
            _pairs_and_loss(g, nl, x, y, p, wns)
    g.close()
