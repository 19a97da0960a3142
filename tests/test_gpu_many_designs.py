"""Batches of hundreds of designs of very uneven size: each instance's summary
and paths are those of a graph of its own, bit for bit (an instance's endpoints
are summed in the same parts and order whatever else is in the batch)."""
import numpy as np
import pytest
import torch

from paper_2503_11674_amd import netgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,n", [(40, -1), (300, 2), (700, -1)])
def test_instances_equal_graphs_of_their_own(library, count, n):
    from paper_2503_11674_amd import tdp
    kinds = []
    for i, (cells, ff) in enumerate([(30, 0.3), (70, 0.2), (400, 0.15), (30_000, 0.5), (9000, 0.4), (55, 0.6)]):
        cfg = netgen.NetlistConfig(f"m{i}", cells, ff_frac=ff, depth=3 if cells < 100 else 6, fanin_lo=1, fanin_hi=4, fanout_cap=12,
                                   die=15.0 * cells ** 0.5, seed=i + 1)
        nl = netgen.make_netlist(cfg)
        nl["clock_period"] = np.float32(150.0 + 20 * i)
        kinds.append(nl)
    rng = np.random.default_rng(count)
    which = rng.choice(len(kinds), count, p=[0.35, 0.3, 0.2, 0.02, 0.03, 0.1])
    which[[3, count - 1]] = 3  # a large one among the first, one at the end
    k, K = 2, 60
    own = []
    for nl in kinds:
        g = tdp.TimingGraph(nl, library, max_paths=K, max_k=k)
        g.sta_update(*[torch.tensor(nl[a], device="cuda") for a in ("x", "y")])
        s = g.summary()
        if n < 0:
            g.report_timing(K)
        else:
            g.extract_paths(n=n, k=k, K=K)
        own.append((s, g.paths()))
        g.close()
    assert any(s[1] < 0 for s, _ in own)
    nls = [kinds[i] for i in which]
    g = tdp.TimingGraph(nls, library, max_paths=K, max_k=k)
    x, y = [torch.tensor(np.concatenate([nl[a] for nl in nls]), device="cuda") for a in ("x", "y")]
    for _ in range(2):
        g.sta_update(x, y)
        w, t, f = g.batch_summary()
    if n < 0:
        g.report_timing(K)
    else:
        g.extract_paths(n=n, k=k, K=K)
    p = g.paths()
    pb, _ = g.batch_offsets()
    inst = np.searchsorted(pb, p["path_ep"], side="right") - 1
    for i, kind in enumerate(which):
        (ws, ts, fs), q = own[kind]
        assert (w[i], t[i], f[i]) == (ws, ts, fs), i
        idx = np.nonzero(inst == i)[0]
        assert len(idx) == q["num_paths"]
        assert np.array_equal(p["path_slack"][idx], q["path_slack"])
        if n >= 0:
            assert np.array_equal(p["path_ep"][idx] - pb[i], q["path_ep"])
            for a, b in zip(idx, range(q["num_paths"])):
                assert np.array_equal(p["path_pins"][p["path_ptr"][a]:p["path_ptr"][a + 1]] - pb[i],
                                      q["path_pins"][q["path_ptr"][b]:q["path_ptr"][b + 1]])
    g.close()


def test_many_designs_take_no_longer_than_few(library):
    """The update of 1,000 designs against 20 of as many cells in all: the least
    of 20 runs each, within a factor of four (the same work, in the same launches)."""
    from paper_2503_11674_amd import tdp
    best = []
    for count in (20, 1000):
        cells = 100_000 // count
        cfg = netgen.NetlistConfig("t", cells, ff_frac=0.15, depth=10, fanin_lo=1, fanin_hi=4, fanout_cap=12,
                                   die=15.0 * cells ** 0.5, seed=1)
        nl = netgen.make_netlist(cfg)
        nl["clock_period"] = np.float32(200.0)
        g = tdp.TimingGraph([nl] * count, library, max_paths=10, max_k=1)
        x, y = [torch.tensor(np.tile(nl[a], count), device="cuda") for a in ("x", "y")]
        runs = []
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.sta_update(x, y)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b))
        best.append(min(runs))
        g.close()
    assert best[1] < 4 * best[0], best
