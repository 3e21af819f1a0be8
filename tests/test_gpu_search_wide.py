"""Searches with windows wider than the staged hit words (2,048 particles): one
search kernel counts every row, wide or not (the launch timing holds it under
both of its names), and the rows are those of the count-only call and of a
brute-force count."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _crowd():
    """A 2-D lattice with one crowded spot: few of its windows are wide."""
    w = I.make_2d(60, 50, 1.0, 0.10)
    rng = np.random.default_rng(4)
    w.pos = np.concatenate([w.pos, rng.uniform(0.4, 0.4 + 2 * w.dx, (2, 2200))], axis=1)
    w.vol = np.full(w.pos.shape[1], w.dx ** 2)
    return w


SETS = {
    "none": (lambda: I.make_2d(600, 400, 1.0, 0.10), 3.0, False),
    "some": (_crowd, 3.0, True),
    "all-2d": (lambda: I.make_2d(60, 600, 1.0, 0.10), 16.0, True),
    "all-3d": (lambda: I.make_sigma3d(24, 24, 24, 0.05), 5.0, True),
}


@pytest.mark.parametrize("name", list(SETS))
def test_one_search(name):
    make, Rs, wide = SETS[name]
    w = make()
    R = Rs * w.dx
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, R, w.kernel, device=DEV, keep_col=False)
    rows = g.row_ptr.clone()
    g.row_ptr.zero_()
    vct.vct_timing_reset()
    vct.vct_timing_enable(True)
    try:
        nnz, staged = vct.vct_neighbors_search(g.nl, g.pos, g._nws)
    finally:
        vct.vct_timing_enable(False)
    ran = {k: v for k, v in vct.vct_timing_read().items() if "k_nb" in k}
    vct.vct_timing_reset()
    assert {k: v[0] for k, v in ran.items()} == {"k_nb_chunk (stage)": 1, "k_nb_chunk (count)": 1}
    assert ran["k_nb_chunk (count)"][1] >= ran["k_nb_chunk (stage)"][1]   # the one launch, timed around the other
    assert staged == (0 if wide else 1) and nnz == g.nnz
    assert torch.equal(g.row_ptr, rows)
    g.row_ptr.zero_()
    nl = vct.vct_nlist.from_buffer_copy(g.nl)
    nl.col16 = None
    assert vct.vct_neighbors(nl, g.pos, 0, 0, g._nws) == (vct.VCT_OK, nnz)   # the counts alone
    assert torch.equal(g.row_ptr, rows)
    pos = g.pos[:, : g.n].cpu().numpy()
    deg = np.diff(rows.cpu().numpy())
    for i in np.random.default_rng(1).choice(g.n, 40, replace=False):
        d = pos - pos[:, i: i + 1]
        d2 = d[0] * d[0] + d[1] * d[1] + (d[2] * d[2] if w.dim == 3 else 0.0)
        assert deg[i] == np.count_nonzero(d2 < R * R) - 1
