"""The transposed-entry map against its definition: entry col_t[e] of e =
(i, j) lies in row j and holds i.  Rows from the hit words (with the columns'
positions) and from the fill pass (without), windows within one part of the
kernel's LDS and beyond it, with and without the 16-bit offsets."""
import ctypes as C

import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def check(row_ptr, col, col_t):
    rp, col, ct = (t.cpu().numpy().astype(np.int64) for t in (row_ptr, col, col_t))
    n = rp.shape[0] - 1
    row = np.repeat(np.arange(n), np.diff(rp))
    assert ct.min() >= 0 and ct.max() < col.shape[0]
    assert np.array_equal(row[ct], col)   # in row j ...
    assert np.array_equal(col[ct], row)   # ... the entry of i


def sets():
    yield "2d", I.small("bf2d"), 1.0
    yield "2d-wide", I.make_2d(60, 600, 1.0, 0.10), 5.0   # windows beyond one part and beyond the hit words
    for Rs in (1.0, 1.3, 1.45, 1.6):                        # one part, two parts, fill pass
        yield f"3d-{Rs}", I.small("sigma3d"), Rs
    w = I.small("sigma3d")
    rng = np.random.default_rng(3)
    k = rng.choice(w.n, 60, replace=False)
    w.pos[0, k[:30]] += rng.choice([-1.0, 1.0], 30) * 0.7   # outside the box: far from their cells' particles
    extra = np.random.default_rng(8).uniform(0.40, 0.45, (3, 150))   # a crowded corner of one cell
    extra[2] -= 0.25
    w.pos = np.concatenate([w.pos, extra], axis=1)
    w.vol = np.concatenate([w.vol, np.full(150, w.vol[0])])
    yield "3d-uneven", w, 1.0
    yield "one-cell", I.make_2d(5, 3, 1.0, 0.10), 9.0
    yield "3d-thin", I.make_sigma3d(40, 5, 3, 0.05), 1.0


@pytest.mark.parametrize("name,w,Rs", list(sets()), ids=lambda v: v if isinstance(v, str) else "")
def test_transposed_entry_map(name, w, Rs):
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, Rs * w.R, w.kernel, device=DEV)
    check(g.row_ptr, g.col[: g.nnz], g.col_t[: g.nnz])
    # without the 16-bit offsets: from the rows of the search, and of the fill pass
    for reuse in (0, 1):
        col_t = torch.full_like(g.col_t, -7)
        nl = vct.vct_nlist.from_buffer_copy(g.nl)
        nl.col16, nl.col_t = None, C.c_void_p(col_t.data_ptr())
        st, nnz = vct.vct_neighbors(nl, g.pos, g.nnz, reuse, g._nws)
        assert st == vct.VCT_OK and nnz == g.nnz
        assert torch.equal(col_t[: g.nnz], g.col_t[: g.nnz])
