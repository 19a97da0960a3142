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


@pytest.mark.parametrize("model", [0, 1, 2])
@pytest.mark.parametrize("part", ["forward", "backward"])
def test_smoothed_sweeps_that_gave_up_are_reported(library, model, part):
    """The value or the gradients are not numbers, and the next call that waits
    for results says so once, though an update lies between."""
    from paper_2503_11674_amd import tdp
    nl = _design(library, 3000, 40)
    g = tdp.TimingGraph(nl, dict(library, net_model=model), max_paths=100, max_k=1)
    x, y = _xy(nl)
    one = torch.ones((), dtype=torch.float64, device="cuda")

    def bwd():
        gx, gy = torch.zeros_like(x), torch.zeros_like(y)
        g.stns_bwd(one, gx, gy)
        return torch.stack((gx, gy))

    g.sta_update(x, y)
    want = g.summary()
    value, grad = float(g.stns_fwd(x, y, 10.0)), bwd()
    assert np.isfinite(value) and bool(torch.isfinite(grad).all())
    fixed = torch.tensor(nl["cell_fixed"], device="cuda").bool()
    for readers in ((g.summary, g.paths_count), (g.batch_summary, g.summary), (g.paths_count, g.summary)):
        g.extract_paths(n=-1, k=1)
        if part == "backward":
            assert float(g.stns_fwd(x, y, 10.0)) == value
        g.set_tuning(spin_log2=1)
        if part == "forward":
            assert np.isnan(float(g.stns_fwd(x, y, 10.0)))
        assert bool(torch.isnan(bwd()[:, ~fixed]).all())
        g.set_tuning(spin_log2=20)
        g.sta_update(x, y)
        g.extract_paths(n=-1, k=1)
        _reports(tdp, readers[0])
        readers[0]()
        readers[1]()
        assert g.summary() == want
        assert float(g.stns_fwd(x, y, 10.0)) == value and torch.equal(bwd(), grad)
    g.close()


def _all_results(g, x, y, k):
    """Everything that the four sweeps make."""
    out = [v.cpu().numpy() for v in g.export().values()]
    g.extract_paths(n=-1, k=k)
    p = g.paths()
    out += [p[q] for q in ("path_ptr", "path_pins", "path_slack")]
    value = g.stns_fwd(x, y, 10.0)
    for _ in range(2):
        gx, gy = torch.zeros_like(x), torch.zeros_like(y)
        g.stns_bwd(torch.ones((), dtype=torch.float64, device="cuda"), gx, gy)
        out += [gx.cpu().numpy(), gy.cpu().numpy()]
    return out + [float(value), g.summary()]


@pytest.mark.parametrize("cells,depth,k,prec,fanin_hi", [(300, 40, 1, "f32", 4), (5000, 60, 3, "f32", 4),
                                                         (5000, 60, 8, "f32", 20), (20_000, 50, 20, "f32", 4),
                                                         (3000, 60, 1, "f64", 4)])
def test_sweeps_by_tickets(library, cells, depth, k, prec, fanin_hi):
    """A budget so small that waves soon leave their fixed shares and large
    enough to end by tickets: the results are the same bits, and no error."""
    from paper_2503_11674_amd import tdp
    cfg = netgen.NetlistConfig("t", cells, ff_frac=0.15, depth=depth, fanin_lo=1, fanin_hi=fanin_hi, fanout_cap=20,
                               die=15.0 * cells ** 0.5, seed=9)
    nl = with_clock(netgen.make_netlist(cfg), library, 0.3)
    x, y = _xy(nl)
    for model in (0, 2):
        outs = []
        for form in ("levels", "shares", "tickets"):
            g = tdp.TimingGraph(nl, dict(library, net_model=model), precision=prec, max_paths=20_000, max_k=k)
            if form == "levels":
                g.set_tuning(sweep_mode=0)
            elif form == "tickets" and prec == "f32":
                g.set_tuning(spin_log2=12)
            for i in range(3):
                if i == 1:
                    g.sta_update_arrivals(x, y)
                    g.sta_update_required()
                    g.sta_update_required()
                else:
                    g.sta_update(x, y)
                outs.append(_all_results(g, x, y, k))
            g.close()
        for o in outs[1:]:
            for a, b in zip(outs[0], o):
                assert np.array_equal(a, b)


@pytest.mark.parametrize("graphs,k", [(3, 16), (8, 10), (16, 1)])
def test_sweeps_of_many_graphs_at_once(library, graphs, k):
    """Graphs on streams of their own, more than their grids fit on the GPU."""
    from paper_2503_11674_amd import tdp
    work = []
    for i in range(graphs):
        nl = _design(library, 20_000 + 700 * i, 40, seed=i)
        g = tdp.TimingGraph(nl, library, max_paths=5000, max_k=k)
        x, y = _xy(nl)
        g.sta_update(x, y)
        want = _all_results(g, x, y, k)
        gx, gy = torch.zeros_like(x), torch.zeros_like(y)
        work.append((g, x, y, gx, gy, want, torch.cuda.Stream()))
    one = torch.ones((), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for _ in range(30):
        for g, x, y, gx, gy, _, s in work:
            with torch.cuda.stream(s):
                g.sta_update(x, y)
                g.extract_paths(n=-1, k=k)
                g.stns_fwd(x, y, 10.0)
                g.stns_bwd(one, gx, gy)
    torch.cuda.synchronize()
    for g, x, y, _, _, want, s in work:
        with torch.cuda.stream(s):
            g.summary()
        torch.cuda.synchronize()
        for a, b in zip(want, _all_results(g, x, y, k)):
            assert np.array_equal(a, b)
        g.close()


@pytest.mark.parametrize("bits", [-1, -2, 0x7FFFFFFF, 0x7FC00000, 0x7F800000])
@pytest.mark.parametrize("k,prec", [(1, "f32"), (4, "f32"), (1, "f64")])
def test_positions_that_are_not_finite_spoil_their_own_instance(library, bits, k, prec):
    """NaNs of every payload, the words' "not yet" among them, and infinities in
    one design of a batch: no wait runs out, and the others' results stand."""
    from paper_2503_11674_amd import tdp
    nls = [_design(library, n, 12, seed=n) for n in (300, 700, 500)]
    if prec == "f64":
        nls = nls[1:2]
    g = tdp.TimingGraph(nls if len(nls) > 1 else nls[0], library, precision=prec, max_paths=100, max_k=k)
    x, y = _xy(*nls)
    g.sta_update(x, y)
    want = g.batch_summary()
    first = g.batch_offsets()[1][1] if len(nls) > 1 else 0
    bad = [a.clone() for a in (x, y)]
    for a in bad:
        a.view(torch.int32)[first:first + nls[-1 if prec == "f64" else 1]["num_cells"]:3] = bits
    g.sta_update(*bad)
    got = g.batch_summary()
    for a, b in zip(want, got):
        for i in (0, 2) if len(nls) > 1 else ():
            assert a[i] == b[i]
    with pytest.raises(tdp.TdpError) as e:
        g.summary()
    assert e.value.status == 1
    g.sta_update(x, y)
    for a, b in zip(want, g.batch_summary()):
        assert np.array_equal(a, b)
    g.close()


def test_an_ordering_that_gave_up(library):
    """Barriers of an ordering over several workgroups with a budget of a few
    polls: the call's paths are right or reported, and the next ones are right."""
    from paper_2503_11674_amd import tdp
    cfg = netgen.NetlistConfig("o", 40_000, ff_frac=0.5, depth=6, fanin_lo=1, fanin_hi=4, fanout_cap=12, die=3000.0,
                               seed=3)
    nl = with_clock(netgen.make_netlist(cfg), library, 0.4)
    g = tdp.TimingGraph(nl, library, max_paths=100_000, max_k=4)
    x, y = _xy(nl)
    names = ("path_ptr", "path_pins", "path_ep", "path_rank", "path_slack")
    calls = [(-1, 4), (3000, 1), (10 ** 9, 4), (2000, 2)]
    want = []
    g.set_tuning(sweep_mode=0)
    g.sta_update(x, y)
    for n, k in calls:
        g.extract_paths(n=n, k=k)
        want.append(g.paths())
    for rnd in range(6):
        for (n, k), w in zip(calls, want):
            g.set_tuning(spin_log2=1 + rnd % 3, sweep_mode=0)
            g.sta_update(x, y)
            g.extract_paths(n=n, k=k)
            g.pairs_update()
            try:
                p = g.paths()
            except tdp.TdpError as e:
                assert e.status == DEVICE_ERROR
            else:
                assert all(np.array_equal(p[q], w[q]) for q in names)
            g.set_tuning(spin_log2=20, sweep_mode=0)
            g.sta_update(x, y)
            g.extract_paths(n=n, k=k)
            p = g.paths()
            assert all(np.array_equal(p[q], w[q]) for q in names)
    g.close()


def test_an_incremental_update_after_a_give_up(library):
    """It starts from values that are not right, so the error stays until a full
    update."""
    from paper_2503_11674_amd import tdp
    nl = _design(library, 3000, 12)
    g = tdp.TimingGraph(nl, library, max_paths=100, max_k=4)
    x, y = _xy(nl)
    moved = torch.nonzero(torch.tensor(nl["cell_fixed"]) == 0)[:3, 0].to(torch.int32).cuda()
    for spin in (4, 1):
        g.set_tuning(spin_log2=20, sweep_mode=1)
        g.sta_update(x, y)
        want = g.summary()
        g.sta_update_arrivals_incremental(x, y, moved)
        g.sta_update_required()
        assert g.summary() == want
        g.set_tuning(spin_log2=spin, sweep_mode=2)
        g.sta_update(x, y)
        g.set_tuning(spin_log2=20, sweep_mode=1)
        for _ in range(2):
            g.sta_update_arrivals_incremental(x, y, moved)
            g.sta_update_required()
            _reports(tdp, g.summary)
            _reports(tdp, g.batch_summary)
        g.sta_update(x, y)
        assert g.summary() == want
    g.close()


@pytest.mark.parametrize("between", ["rise_fall", "incremental"])
@pytest.mark.parametrize("give_ups", [1, 2, 3, 4])
def test_give_ups_with_other_updates_between(library, between, give_ups):
    """Records of the last good pass, four numbers old after three passes that
    gave up, are not taken for the new pass's, also where another kind of
    update has cleared the error word between them."""
    from paper_2503_11674_amd import tdp
    nl = _design(library, 3000, 12)
    k = 4
    sets = [[torch.tensor(a, device="cuda") for a in netgen.jitter_positions(nl, 30.0, s)] for s in (1, 2)]
    moved = torch.arange(3, dtype=torch.int32, device="cuda")

    def result(g):
        g.extract_paths(n=-1, k=k)
        p = g.paths()
        return g.summary(), [p[key] for key in ("path_ptr", "path_pins", "path_ep", "path_slack")]

    fresh = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
    fresh.set_tuning(sweep_mode=0)
    fresh.sta_update(*sets[1])
    want = result(fresh)
    fresh.close()
    g = tdp.TimingGraph(nl, library, max_paths=4000, max_k=k)
    g.rf_setup(netgen.make_rf_library(library))
    g.sta_update(*sets[0])
    for _ in range(give_ups):
        g.set_tuning(spin_log2=4, sweep_mode=2)
        g.sta_update(*sets[0])
        if between == "rise_fall":
            g.sta_update_rf(*sets[0])
        else:
            g.sta_update_arrivals_incremental(*sets[0], moved)
    g.set_tuning(spin_log2=20, sweep_mode=1)
    g.sta_update(*sets[1])
    got = result(g)
    assert got[0] == want[0]
    for a, b in zip(got[1], want[1]):
        assert np.array_equal(a, b)
    g.close()
