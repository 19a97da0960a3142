"""The pair set, its per-cell lists and the endpoint summary where their
launches' tiles end: fewer sinks than a tile, a ragged second one, and designs
whose tiles hold 16 sinks a thread; endpoints in one part and in many, and
instances of uneven size.

Pairs are the oracle's rule applied to the extraction's own paths: weights to
1e-4 (single-precision slacks against the oracle's double), the losses'
gradients to 1e-4 of the sum of absolute terms at a cell.  The summary is
exact but for the order of a double sum."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2503_11674_amd import netgen
from tests.conftest import with_clock
from tests.test_gpu_parity import _p2p_abs_scale

pytestmark = pytest.mark.gpu


def _design(library, cells, seed=5, ff_frac=0.12, depth=9):
    cfg = netgen.NetlistConfig("p", cells, ff_frac=ff_frac, depth=depth, fanout_cap=12, die=20.0 * cells ** 0.5,
                               seed=seed)
    nl = with_clock(netgen.make_netlist(cfg), library, 0.2)
    fixed = np.zeros(nl["num_cells"], np.uint8)
    fixed[::7] = 1
    return dict(nl, cell_fixed=fixed)


def _xy(nl, seed=None):
    x, y = (nl["x"], nl["y"]) if seed is None else netgen.jitter_positions(nl, 15.0, seed)
    return x, y, torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda")


@pytest.mark.parametrize("cells,prec", [(400, "f32"), (1800, "f32"), (3600, "f64"), (950_000, "f32")])
def test_pairs_and_their_lists(library, cells, prec):
    from paper_2503_11674_amd import tdp
    nl = _design(library, cells)
    E = len(ref.endpoint_pins(nl))
    k = 3
    g = tdp.TimingGraph(nl, library, precision=prec, max_paths=E * k, max_k=k)
    if cells > 100_000:
        assert g.num_sinks > 512 * 4096
    ps = ref.PairState(nl["num_pins"])
    for i, (rule, K) in enumerate([(0, E), (0, 40), (1, E * k), (1, 25), (0, E * k)]):
        x, y, xd, yd = _xy(nl, 20 + i)
        g.sta_update(xd, yd)
        g.extract_paths(n=-1, k=k, K=K)
        g.pairs_update(rule=rule, w0=10.0, w1=0.2)
        ref.pairs_update(ps, g.paths(), g.summary()[0], rule=rule)
        w, member = g.pairs_export()
        print("round", i, rule, K, int(member.sum()), flush=True)
        assert member.any() and np.array_equal(member.astype(bool), ps.in_p.astype(bool))
        sinks = np.nonzero(member)[0]
        assert np.allclose(w[sinks], ps.w[sinks], rtol=1e-4)
        gx = torch.zeros(nl["num_cells"], device="cuda")
        gy = torch.zeros_like(gx)
        loss = float(g.p2p_loss_fwd(xd, yd))
        g.p2p_loss_bwd(xd, yd, torch.ones((), dtype=torch.float64, device="cuda"), gx, gy)
        want, wx, wy = ref.p2p(dict(nl, x=x, y=y), sinks, w[sinks].astype(np.float64))
        scale = _p2p_abs_scale(dict(nl, x=x, y=y), sinks, w[sinks])
        assert abs(loss - want) <= 1e-4 * abs(want)
        assert np.all(np.abs(gx.cpu().numpy() - wx) <= 1e-4 * scale + 1e-6)
        assert np.all(np.abs(gy.cpu().numpy() - wy) <= 1e-4 * scale + 1e-6)
    g.close()


@pytest.mark.parametrize("cells", [(9,), (2000,), (60_000,), (400, 30_000, 70, 5000)])
def test_endpoint_summary(library, cells):
    """Parts of an instance's endpoints: none, one, ragged, many."""
    from paper_2503_11674_amd import tdp
    nls = [_design(library, c, seed=3 + i, ff_frac=0.4, depth=3) for i, c in enumerate(cells)]
    for nl in nls:
        nl["clock_period"] = nls[0]["clock_period"]
    g = tdp.TimingGraph(nls if len(nls) > 1 else nls[0], library, max_paths=10, max_k=1)
    x, y = (torch.tensor(np.concatenate([nl[c] for nl in nls]), device="cuda") for c in "xy")
    for _ in range(2):
        g.sta_update(x, y)
        slack = g.export()["slack"].cpu().numpy().astype(np.float64)
        got = g.batch_summary() if len(nls) > 1 else [[v] for v in g.summary()]
        base = 0
        for i, nl in enumerate(nls):
            s = slack[base + ref.endpoint_pins(nl)]
            base += nl["num_pins"]
            s = s[s < 0]
            assert got[0][i] == (s.min() if len(s) else 0.0) and got[2][i] == len(s)
            assert abs(got[1][i] - s.sum()) <= 1e-12 * abs(s.sum())
    g.close()
