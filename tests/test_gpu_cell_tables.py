"""The cell and chunk tables against their definitions: cell_start over grids
at the edges of the scan's forms (one work-group, tiles that add up their own
offsets, a scan of the tile sums), and the chunk table of columns with none,
few and more than sixteen chunks."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("grid", [(1, 1), (1, 7), (128, 127), (128, 128), (145, 113), (2048, 9), (3, 6827),
                                  (4096, 4096), (4096, 4101)], ids=str)
def test_cell_starts(grid):
    nx, nz = grid
    n, R = 5003, 1.0
    lo, hi = (0.0, 0.0), (nx * 1.00001, nz * 1.00001)   # cells just wider than R
    ncell, dims = vct.vct_grid_dims(2, lo, hi, R)
    assert dims[:2] == grid and ncell == nx * nz
    pos = np.random.default_rng(1).uniform(0.0, 1.0, (2, n)) * np.asarray(hi)[:, None]
    p = torch.as_tensor(pos, device=DEV)
    perm = torch.empty(n, dtype=torch.int32, device=DEV)
    ps = torch.empty_like(p)
    cs = torch.empty(ncell + 1, dtype=torch.int64, device=DEV)
    ws = torch.empty(vct.lib().vct_build_cells_workspace_size(2, n, ncell), dtype=torch.uint8, device=DEV)
    vct.vct_build_cells(2, n, p, lo, hi, R, perm, ps, cs, ncell, ws)
    co = [np.clip(np.floor(pos[a] * (float(grid[a]) / hi[a])), 0, grid[a] - 1).astype(np.int64) for a in range(2)]
    key = co[0] * nz + co[1]
    start = np.zeros(ncell + 1, dtype=np.int64)
    start[1:] = np.cumsum(np.bincount(key, minlength=ncell))
    assert np.array_equal(cs.cpu().numpy(), start)
    assert np.array_equal(perm.cpu().numpy(), np.lexsort((np.arange(n), key)))


def chunk_sets():
    yield "2d-tall", I.make_2d(24, 900, 1.0, 0.10)         # 42 chunks a column
    yield "2d-17", I.make_2d(31, 350, 1.0, 0.05)           # 16 and 17 chunks a column
    yield "3d", I.small("sigma3d")
    w = I.small("sigma3d")
    far = np.all([w.pos[0] > 0.4, w.pos[1] > 0.3], axis=0)   # columns without particles
    w.pos, w.vol = np.ascontiguousarray(w.pos[:, ~far]), w.vol[~far]
    yield "3d-gaps", w


@pytest.mark.parametrize("name,w", list(chunk_sets()), ids=lambda v: v if isinstance(v, str) else "")
def test_chunk_table(name, w):
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=False)
    nz = g.dims[w.dim - 1]
    cs = g.cell_start.cpu().numpy()
    cell = np.searchsorted(cs, np.arange(w.pos.shape[1]), side="right") - 1   # of every sorted particle
    col, z = cell // nz, cell % nz
    ncols = g.ncell // nz
    first = cs[:-1].reshape(ncols, nz)[:, 0]
    count = np.diff(np.concatenate([first, [cs[-1]]]))
    nch = -(-count // 64)
    off = np.concatenate([[0], np.cumsum(nch)])
    assert np.array_equal(g.chunk_off.cpu().numpy(), off)
    start = np.concatenate([first[c] + 64 * np.arange(nch[c]) for c in range(ncols)]).astype(np.int64)
    end = np.minimum(start + 64, np.repeat(first + count, nch)) - 1
    assert np.array_equal(g.chunk_start.cpu().numpy()[: off[-1] + 1], np.concatenate([start, [cs[-1]]]))
    info = np.stack([col[start], z[start], z[end], np.zeros_like(start)], 1)
    assert np.array_equal(g.chunk_info.cpu().numpy()[: off[-1]], info)
    assert nch.max() > (16 if name.startswith("2d") else 1) and (name != "3d-gaps" or nch.min() == 0)
