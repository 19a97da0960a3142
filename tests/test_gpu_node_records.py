"""The node records (hops, chain depths, deviation lists) that both forward
sweeps make, at the sizes where their lane groups, list waves' turns and
published words can go wrong: every list width, levels that are no multiple
of a turn, cells with more inputs than lanes, passes in a row under the same
and under changing sweep forms, and a pass after sweeps that gave up.

Arrivals, paths and their order are bitwise those of the per-level form, and
the paths match the oracle's: a deviation's cost is one subtraction of two
arrivals, the same in every form."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_11674_amd import netgen
from tests.bruteforce import Graph
from tests.comparator import compare_paths
from tests.conftest import with_clock

pytestmark = pytest.mark.gpu

PATHS = ("path_ptr", "path_pins", "path_ep", "path_rank", "path_slack")


def _design(library, cells=611, depth=13, fanin_hi=4, seed=3):
    cfg = netgen.NetlistConfig("n", cells, ff_frac=0.15, depth=depth, fanin_lo=1, fanin_hi=fanin_hi,
                               fanout_cap=12 if fanin_hi <= 20 else 60,
                               die=700.0, seed=seed)
    return with_clock(netgen.make_netlist(cfg), library, 0.4)


def _xy(nl, seed=None):
    x, y = (nl["x"], nl["y"]) if seed is None else netgen.jitter_positions(nl, 20.0, seed)
    return torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda")


def _result(g, k):
    g.extract_paths(n=-1, k=k)
    p = g.paths()
    return {**{q: v.cpu().numpy() for q, v in g.export().items()}, **{q: p[q] for q in PATHS}}


def _same(a, b):
    for q in a:
        assert np.array_equal(a[q], b[q]), q


# (the sizes put the last turn of a level at every remainder of 8, 4 and 2)
@pytest.mark.parametrize("k,fanin_hi", [(1, 4), (2, 4), (3, 12), (7, 4), (8, 12), (11, 4), (16, 20), (20, 4), (32, 40)])
def test_list_widths_and_wide_cells(library, k, fanin_hi):
    from paper_2503_11674_amd import tdp
    nl = _design(library, fanin_hi=fanin_hi, cells=600 + 7 * k)
    st = ref.sta(nl, library)
    E = len(ref.endpoint_pins(nl))
    outs = []
    for mode in (0, 1):
        g = tdp.TimingGraph(nl, library, max_paths=E * k, max_k=k)
        g.set_tuning(sweep_mode=mode)
        g.sta_update(*_xy(nl))
        outs.append(_result(g, k))
        p = g.paths()
        g.close()
    _same(*outs)
    rp = ref.extract(nl, library, st, n=-1, k=k)
    assert p["num_paths"] == rp["num_paths"]
    res = compare_paths(p, rp, st, Graph(nl), k)
    assert res["missing"] == 0 and res["extra"] == 0
    assert res["pinned_ok"] == res["pinned"] and res["unpinned_ok"] == res["unpinned"]


@pytest.mark.parametrize("prec,k,wide_net", [("f64", 1, False), ("f64", 5, False), ("f64", 1, True), ("f32", 5, True)])
def test_sweeps_of_graphs_without_a_sweep_mode(library, prec, k, wide_net):
    """Double precision, or a net wider than a chunk: the graph's own choice
    of sweeps against one launch per level."""
    from paper_2503_11674_amd import tdp
    nl = _design(library)
    if wide_net:  # the first nets' sinks all on the first port's net
        nl = dict(nl, net_ptr=nl["net_ptr"].copy(), net_pins=nl["net_pins"].copy())
        ptr, pins = nl["net_ptr"], nl["net_pins"]
        port = int(np.nonzero(nl["pin_cell"][pins[ptr[:-1]]] < 0)[0][0])
        drv = pins[ptr[:-1]]
        sinks = [list(pins[a + 1:b]) for a, b in zip(ptr[:-1], ptr[1:])]
        for n in range(len(drv)):
            if n != port and len(sinks[port]) < 90 and nl["pin_cell"][drv[n]] < 0:
                sinks[port] += sinks[n]
                sinks[n] = []
        assert len(sinks[port]) > 63
        ptr[1:] = np.cumsum([1 + len(s) for s in sinks])
        nl["net_pins"] = np.concatenate([[d] + s for d, s in zip(drv, sinks)]).astype(np.int32)
    outs = []
    for levels in (True, False):
        g = tdp.TimingGraph(nl, library, precision=prec, max_paths=4000, max_k=k)
        if levels:
            g.set_tuning(sweep_mode=0)
        for s in (5, 6, None):
            g.sta_update(*_xy(nl, s))
        outs.append(_result(g, k))
        g.close()
    _same(*outs)


@pytest.mark.parametrize("k", [1, 10])
def test_passes_in_a_row(library, k):
    """More passes than a tag has values, under one form and under changing
    ones, rise / fall and incremental passes between them, and passes after
    sweeps that gave up: each equal to a fresh graph's."""
    from paper_2503_11674_amd import tdp
    nl = _design(library)
    rf = netgen.make_rf_library(library)
    fresh = {}
    for s in (11, 12):
        g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
        g.set_tuning(sweep_mode=0)
        g.sta_update(*_xy(nl, s))
        fresh[s] = _result(g, k)
        g.close()
    g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
    g.rf_setup(rf)
    for i, mode in enumerate((1, 1, 1, 1, 1, 0, 1, 3, 3, 3, 1, 2, 2, 2, 2, 1, 0, 0, 0, 1)):
        s = 11 + i % 2
        g.set_tuning(spin_log2=4 if mode == 2 else 20, sweep_mode=mode)
        g.sta_update(*_xy(nl, s))
        if mode == 2:
            with pytest.raises(tdp.TdpError):
                g.summary()
            continue
        _same(_result(g, k), fresh[s])
        if i % 3 == 1:
            for _ in range(3):
                g.sta_update_rf(*_xy(nl, s))
        if i == 6:
            g.sta_update(*_xy(nl, s))
            g.sta_update_arrivals_incremental(*_xy(nl, 23 - s), torch.arange(g.num_cells, dtype=torch.int32, device="cuda"))
            g.sta_update_required()
            _same(_result(g, k), fresh[23 - s])
    g.close()


def test_replayed_update(library):
    """A captured update replayed with other work between the replays."""
    from paper_2503_11674_amd import tdp
    nl = _design(library)
    g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=4)
    x, y = _xy(nl)
    g.sta_update(x, y)
    g.extract_paths(n=-1, k=4)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.sta_update(x, y)
        g.extract_paths(n=-1, k=4)
    for s in (21, 22, 23, 24, 25, 26):
        xs, ys = _xy(nl, s)
        ref_g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=4)
        ref_g.sta_update(xs, ys)
        want = _result(ref_g, 4)
        ref_g.close()
        x.copy_(xs)
        y.copy_(ys)
        graph.replay()
        p = g.paths()
        _same({**{q: v.cpu().numpy() for q, v in g.export().items()}, **{q: p[q] for q in PATHS}}, want)
        if s % 2:  # an eager pass at other positions between two replays
            g.sta_update(*_xy(nl, 50 + s))
            torch.cuda.synchronize()
    g.close()


@pytest.mark.parametrize("modes", [(0, 0, 0, 1), (3, 3, 3, 1, 3, 0, 3, 1), (1, 0, 0, 0, 1, 3, 3, 3, 1),
                                   (1, 1) + 7 * (0,) + (1, 2, 0, 0, 0, 1)])
@pytest.mark.parametrize("sets", [3, 5])
def test_grid_passes_after_passes_by_level(library, modes, sets):
    """Three and seven passes by level between two grid passes, and before a
    new graph's first: the words that only grid passes write are then four or
    eight passes old, and of other positions."""
    from paper_2503_11674_amd import tdp
    nl = _design(library)
    k = 10
    fresh = []
    for s in range(sets):
        g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
        g.set_tuning(sweep_mode=0)
        g.sta_update(*_xy(nl, 31 + s))
        fresh.append(_result(g, k))
        g.close()
    g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
    for i, mode in enumerate(modes):
        g.set_tuning(spin_log2=4 if mode == 2 else 20, sweep_mode=mode)
        g.sta_update(*_xy(nl, 31 + i % sets))
        if mode != 2:
            _same(_result(g, k), fresh[i % sets])
    g.close()


def test_replays_between_passes_by_level(library):
    """A captured grid pass replayed after every three passes by level."""
    from paper_2503_11674_amd import tdp
    nl = _design(library)
    k = 10
    g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
    x, y = _xy(nl)
    g.sta_update(x, y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.sta_update(x, y)
    for r in range(5):
        g.set_tuning(sweep_mode=0)
        for s in range(3):
            g.sta_update(*_xy(nl, 60 + 3 * r + s))
        want = _result(g, k)
        _same(want, _fresh(nl, library, 62 + 3 * r, k))
        for a, b in zip((x, y), _xy(nl, 80 + r)):
            a.copy_(b)
        graph.replay()
        _same(_result(g, k), _fresh(nl, library, 80 + r, k))
    g.close()


def _fresh(nl, library, seed, k):
    from paper_2503_11674_amd import tdp
    g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
    g.set_tuning(sweep_mode=0)
    g.sta_update(*_xy(nl, seed))
    out = _result(g, k)
    g.close()
    return out


@pytest.mark.parametrize("prec,k", [("f64", 1), ("f64", 5), ("f32", 5)])
def test_a_graphs_own_choice_can_be_had_back(library, prec, k):
    """Mode 4 after another one, and by the autotuner: results as by level, and
    the choice it reports is one that can be set."""
    from paper_2503_11674_amd import tdp
    nl = _design(library, cells=900 + k)
    g = tdp.TimingGraph(nl, library, precision=prec, max_paths=4000, max_k=k)
    g.set_tuning(sweep_mode=0)
    x, y = _xy(nl)
    g.sta_update(x, y)
    want = _result(g, k)
    if prec == "f64":
        with pytest.raises(tdp.TdpError):
            g.set_tuning(sweep_mode=1)
    g.set_tuning(sweep_mode=4)
    g.sta_update(x, y)
    _same(_result(g, k), want)
    g.set_tuning(sweep_mode=0)
    ch = g.autotune(x, y, n=-1, k=k, reps=5)
    assert ch["sweep_mode"] in ((0, 4) if prec == "f64" else (0, 1, 3))
    _same(_result(g, k), want)
    g.set_tuning(sweep_mode=ch["sweep_mode"])
    assert g.autotune(x, y, n=-1, k=k, reps=5) == ch
    _same(_result(g, k), want)
    with pytest.raises(tdp.TdpError):
        g.set_tuning(sweep_mode=5)
    g.close()
