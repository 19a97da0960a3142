"""The density's bin gathers where their strips, lanes and crowded rows end:
every radius, grids of one to a few strips either way, rows and windows at the
sizes from which a workgroup sums a bin, everything in one bin; against the
oracle with the bounds of the placement tests (weights and their products in
single precision, sums in double)."""
import numpy as np
import pytest
import torch

from paper_2503_11674_amd import netgen
from tests.test_gpu_placement import _check_density

pytestmark = pytest.mark.gpu


def _graph(library, cells):
    from paper_2503_11674_amd import tdp
    nl = netgen.make_netlist(netgen.NetlistConfig("w", cells, ff_frac=0.2, depth=3, fanout_cap=12, die=500.0, seed=4))
    nl["cell_fixed"] = (np.arange(nl["num_cells"]) % 9 == 0).astype(np.uint8)
    return nl, tdp.TimingGraph(nl, library, max_paths=10, max_k=1)


@pytest.mark.parametrize("gx,gy", [(64, 10), (65, 11), (63, 9), (130, 33), (17, 257)])
@pytest.mark.parametrize("R", range(9))
def test_every_radius_and_ragged_grids(library, gx, gy, R):
    nl, g = _graph(library, 3000)
    rng = np.random.default_rng(gx + R)
    area = rng.uniform(1.0, 6.0, nl["num_cells"]).astype(np.float32)
    grid = dict(x0=0.0, y0=0.0, bw=4.0, bh=2.0, gx=gx, gy=gy, R=R, target=0.4)
    g.density_setup(grid, area)
    x = rng.uniform(-4.0, 4.0 * gx + 4.0, nl["num_cells"]).astype(np.float32)
    y = rng.uniform(-4.0, 2.0 * gy + 4.0, nl["num_cells"]).astype(np.float32)
    _check_density(g, nl, x, y, area, grid, 0.4)
    g.close()


@pytest.mark.parametrize("row", [63, 64, 65, 512, 513])
@pytest.mark.parametrize("R", [0, 3, 4, 6])
def test_crowded_rows_and_windows(library, row, R):
    """`row` cells in one row of bins, in one bin, and over a window's rows."""
    nl, g = _graph(library, 2000)
    n = nl["num_cells"]
    area = np.full(n, 3.0, np.float32)
    grid = dict(x0=0.0, y0=0.0, bw=4.0, bh=4.0, gx=72, gy=40, R=R, target=0.5)
    g.density_setup(grid, area)
    rng = np.random.default_rng(row)
    x = rng.uniform(0.0, 60.0, n).astype(np.float32)
    y = rng.uniform(0.0, 60.0, n).astype(np.float32)
    x[:row] = 200.0 + rng.uniform(0.0, 4.0 * max(R, 1), row)
    y[:row] = 81.25
    x[row:2 * row if row < 500 else row + 400] = 121.25
    y[row:2 * row if row < 500 else row + 400] = 121.25
    _check_density(g, nl, x, y, area, grid, 0.5)
    x[:] = 101.5
    y[:] = 50.25
    _check_density(g, nl, x, y, area, grid, 0.5)
    g.close()


@pytest.mark.parametrize("gx,gy", [(182, 181), (181, 181)])  # 32,942 and 32,761 bins
def test_rows_that_are_almost_crowded_on_average(library, gx, gy):
    """Many bins with rows of 40 to 90 cells: which rows make a bin crowded
    depends on the mean and on the number of bins."""
    nl, g = _graph(library, 300_000)
    n = nl["num_cells"]
    area = np.full(n, 2.0, np.float32)
    grid = dict(x0=0.0, y0=0.0, bw=4.0, bh=4.0, gx=gx, gy=gy, R=3, target=0.5)
    g.density_setup(grid, area)
    rng = np.random.default_rng(gx)
    x = rng.uniform(0.0, 4.0 * gx, n).astype(np.float32)
    y = rng.uniform(0.0, 4.0 * gy, n).astype(np.float32)
    x[:600], y[:600] = 300.0 + rng.uniform(0.0, 20.0, 600), 305.25
    _check_density(g, nl, x, y, area, grid, 0.5)
    g.close()
