"""Which endpoints an extraction takes and the order of its paths, over the
forms that the selection and the ordering have: the violated endpoints or the
n worst (with ties, more than there are, instances above the size that one
workgroup selects), orderings in one workgroup, by counting, by digits and by
the general sort, cut to K or by a slack limit, single designs and batches.

An endpoint's paths do not depend on which others are taken, so every call has
to give the paths of one call that takes all of them, filtered and sorted here:
equality, no tolerance.  That one call's paths match the oracle's elsewhere."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_11674_amd import netgen
from tests.conftest import with_clock
from tests.test_gpu_placement import _check_density

pytestmark = pytest.mark.gpu

PATHS = ("path_ptr", "path_pins", "path_ep", "path_rank", "path_slack")


def _flat(library):
    """Every arc's delay the same: with no wire, many equal slacks."""
    return dict(library, delay_lut=np.full_like(library["delay_lut"], 8.0))


def _design(library, cells, ff_frac=0.5, depth=4, seed=3, ties=False):
    cfg = netgen.NetlistConfig("o", cells, ff_frac=ff_frac, depth=depth, fanout_cap=12, die=700.0, seed=seed)
    nl = netgen.make_netlist(cfg)
    if ties:
        nl = dict(nl, **{a: np.zeros_like(nl[a]) for a in ("x", "y", "pin_off_x", "pin_off_y")})
    nl = with_clock(nl, library, 0.4)
    if ties:  # between two delays' multiples
        nl["clock_period"] = np.float32(nl["clock_period"] - 12)
    return nl


def _graph(nls, library, k, prec):
    from paper_2503_11674_amd import tdp
    E = sum(len(ref.endpoint_pins(nl)) for nl in nls)
    g = tdp.TimingGraph(nls if len(nls) > 1 else nls[0], library, precision=prec, max_paths=E * k, max_k=k)
    g.sta_update(*(torch.tensor(np.concatenate([nl[c] for nl in nls]), device="cuda") for c in "xy"))
    return g, E


def _lists(p):
    ptr, pins = p["path_ptr"], p["path_pins"]
    return [tuple(pins[a:b]) for a, b in zip(ptr[:-1], ptr[1:])]


def _expected(full, bounds, n, k, K, limit):
    """Rows of `full` (every endpoint's paths, unordered) that a call gives."""
    ep, rank, slack = full["path_ep"], full["path_rank"], full["path_slack"]
    rows = []
    for lo, hi in zip(bounds[:-1], bounds[1:]):
        mine = np.nonzero((ep >= lo) & (ep < hi))[0]
        first = mine[rank[mine] == 0]
        # (the n worst are taken by single-precision slacks in both precisions)
        first = first[np.lexsort((ep[first], slack[first].astype(np.float32)))]
        taken = first[slack[first] < 0] if n < 0 else first[:n]
        keep = mine[np.isin(ep[mine], ep[taken]) & (rank[mine] < k) & (slack[mine] < limit)]
        rows.append(keep[np.lexsort((rank[keep], ep[keep], slack[keep]))][:K])
    return np.concatenate(rows)


CALLS = [  # n, k, K, slack limit; None: all of them
    (-1, 1, None, np.inf), (-1, None, None, np.inf), (0, 1, None, np.inf), (1, None, None, np.inf),
    (63, 2, None, np.inf), (257, None, 100, np.inf), (1000, 2, 1999, np.inf), (10 ** 9, 1, None, np.inf),
    (10 ** 9, None, None, 0.0), (10 ** 9, None, 1, np.inf), (-1, None, 1234, np.inf)]


# 400 endpoints at k = 4: one workgroup; 3,000 at 4: by counting; 3,000 at 8 and
# 8,300 at 4: digits, over several workgroups; double precision: the general sort
@pytest.mark.parametrize("cells,k,prec,ties", [
    ((800,), 4, "f32", False), ((800,), 4, "f64", True), ((6000,), 4, "f32", False), ((6000,), 4, "f32", True),
    ((6000,), 8, "f32", False), ((16600,), 4, "f32", True), ((6000,), 8, "f64", False),
    ((300, 5000, 70, 2100), 4, "f32", True), ((300, 34000, 70), 2, "f32", False), ((300, 2000), 3, "f32", True)])
def test_selection_and_order(library, cells, k, prec, ties):
    library = _flat(library) if ties else library
    nls = [_design(library, c, seed=3 + i, ties=ties) for i, c in enumerate(cells)]
    for nl in nls:
        nl["clock_period"] = nls[0]["clock_period"]
    g, E = _graph(nls, library, k, prec)
    bounds = g.batch_offsets()[0] if len(nls) > 1 else np.array([0, nls[0]["num_pins"]])
    g.extract_paths(n=E, k=k)
    full = g.paths()
    assert full["num_paths"] >= E // 2
    lists = _lists(full)
    if ties:
        assert len(np.unique(full["path_slack"])) < full["num_paths"]
    for n, kk, K, limit in [(E, None, None, np.inf)] + CALLS:
        kk = k if kk is None else kk
        print("call", n, kk, K, limit, flush=True)
        want = _expected(full, bounds, n, kk, E * k if K is None else K, limit)
        g.extract_paths(n=n, k=kk, K=K, slack_limit=float(limit))
        p = g.paths()
        for q in ("path_ep", "path_rank", "path_slack"):
            assert np.array_equal(p[q], full[q][want]), (q, n, kk, K, limit)
        assert _lists(p) == [lists[i] for i in want]
    g.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_more_endpoints_than_one_workgroup_selects(library, prec):
    library = _flat(library)
    nl = _design(library, 134000, ties=True)
    g, E = _graph([nl], library, 4, prec)
    assert E > 1 << 16 and 4 * E > 64 * 4096  # (the sort's columns of counts too)
    bounds = np.array([0, nl["num_pins"]])
    g.extract_paths(n=E, k=4)
    full = g.paths()
    for n, k, K in ((-1, 1, None), (1000, 4, None), (65537, 1, None), (E - 1, 4, 3000), (E + 5, 4, None)):
        want = _expected(full, bounds, n, k, 4 * E if K is None else K, np.inf)
        g.extract_paths(n=n, k=k, K=K)
        p = g.paths()
        for q in ("path_ep", "path_rank", "path_slack"):
            assert np.array_equal(p[q], full[q][want]), (q, n, k, K)
    g.close()


def test_calls_from_a_captured_graph(library):
    """One capture of each ordering, replayed with other work between."""
    nl = _design(library, 6000)
    for k in (1, 4, 8):
        g, E = _graph([nl], library, k, "f32")
        g.extract_paths(n=2000, k=k)
        want = g.paths()
        cg = torch.cuda.CUDAGraph()
        with torch.cuda.graph(cg):
            g.extract_paths(n=2000, k=k)
        for _ in range(3):
            cg.replay()
            torch.cuda.synchronize()
            p = g.paths()
            assert all(np.array_equal(p[q], want[q]) for q in PATHS)
            g.extract_paths(n=-1, k=1)
            torch.cuda.synchronize()
        g.close()


@pytest.mark.parametrize("cells,bins", [(4096, 16), (4097, 40), (300001, 500)])
def test_bins_of_many_cells(library, cells, bins):
    """The density's sort of cells by bin: one tile, a ragged second, and more
    tiles than one workgroup adds up.  (Bin widths that single precision holds
    exactly: a cell on a bin's edge is then in the same bin here and there.)"""
    from paper_2503_11674_amd import tdp
    nl = netgen.make_netlist(netgen.NetlistConfig("b", cells, ff_frac=0.2, depth=3, fanout_cap=12, die=2000.0, seed=9))
    area = np.random.default_rng(1).uniform(2.0, 9.0, nl["num_cells"]).astype(np.float32)
    grid = dict(x0=0.0, y0=0.0, bw=2000.0 / bins, bh=2000.0 / bins, gx=bins, gy=bins, R=2, target=0.9)
    g = tdp.TimingGraph(nl, library, max_paths=100, max_k=1)
    g.density_setup(grid, area)
    _check_density(g, nl, nl["x"], nl["y"], area, grid, 0.9)
    g.close()
