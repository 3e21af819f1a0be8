"""vct_neighbors_search followed by vct_neighbors_rows (what Geometry calls)
against one vct_neighbors call on the same particles: the same tables and
columns, with windows that fit the hit words, with some that do not, and with
an empty set; and the capacity and argument errors of the second call."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("family,Rs", [("bf2d", 1.0), ("sigma3d", 1.0), ("sigma3d", 1.15), ("sigma3d", 1.6)])
@pytest.mark.parametrize("keep_col", [False, True])
def test_two_calls_equal_one(family, Rs, keep_col):
    w = I.small(family)
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, Rs * w.R, w.kernel, device=DEV, keep_col=keep_col)
    t = {k: torch.full_like(getattr(g, k), -1 if k != "col16" else 65535)
         for k in ("chunk_off", "chunk_start", "chunk_info", "chunk_win", "row_ptr", "col16")
         + (("col", "col_t") if keep_col else ())}
    nl = vct.make_nlist(g.dim, g.n, g.ncell, w.lo, w.hi, Rs * w.R, g.cell_start, t["chunk_off"], t["chunk_start"],
                        t["chunk_info"], t["row_ptr"], t.get("col"), t["col16"], chunk_cap=g.nl.chunk_cap,
                        col_t=t.get("col_t"), chunk_win=t["chunk_win"])
    st, nnz = vct.vct_neighbors(nl, g.pos, g.nnz, 0, torch.empty_like(g._nws))
    assert st == vct.VCT_OK and nnz == g.nnz == nl.nnz == g.nl.nnz
    nch = int(g.chunk_off[-1].item())
    widest = int(g.chunk_win[:nch].cpu().numpy()[np.arange(nch), 20 + g.chunk_win[:nch, 0].cpu().numpy()].max())
    assert (widest > 2048) == (Rs == 1.6)
    for k, v in t.items():
        m = {"chunk_start": nch + 1, "chunk_info": nch, "chunk_win": nch}.get(k, v.shape[0])
        mine = getattr(g, k)[:m]
        if k == "chunk_win":   # 30 words hold the window, the ranges past its count are unset
            nr = mine[:, 0].cpu().numpy()
            a, b = mine.cpu().numpy(), v[:m].cpu().numpy()
            used = np.zeros_like(a, dtype=bool)
            used[:, 0] = True
            for r in range(9):
                used[nr > r, 2 + 2 * r] = used[nr > r, 3 + 2 * r] = used[nr > r, 20 + r] = True
            assert np.array_equal(a[used], b[used])
        else:
            assert torch.equal(mine, v[:m]), k


def test_rows_errors():
    w = I.small("bf2d")
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=False)
    nnz, staged = vct.vct_neighbors_search(g.nl, g.pos, g._nws)
    assert nnz == g.nnz

    def status(cap, token, ws=g._nws):
        try:
            return vct.vct_neighbors_rows(g.nl, g.pos, cap, token, ws)
        except vct.VctError as e:
            return e.status

    assert status(nnz - 1, staged) == vct.VCT_E_CAPACITY
    assert status(nnz, 7) == vct.VCT_E_ARG and status(nnz, -1) == vct.VCT_E_ARG
    assert status(nnz, staged, g._nws[:100]) == vct.VCT_E_WORKSPACE
    col16, g.nl.col16 = g.nl.col16, None
    assert status(nnz, staged) == vct.VCT_E_ARG
    g.nl.col16 = col16
    ref = g.col16.clone()
    g.col16.fill_(0)
    assert status(nnz, staged) == vct.VCT_OK and torch.equal(g.col16, ref)
    g.col16.fill_(0)
    assert status(nnz, 0) == vct.VCT_OK and torch.equal(g.col16, ref)   # the fill pass, without the words


def test_empty():
    g = vct.Geometry(np.zeros((2, 0)), np.zeros(0), (0, 0), (1, 1), 0.1, device=DEV, keep_col=True)
    assert g.nnz == 0 and int(g.chunk_off[-1].item()) == 0 and g.row_ptr.tolist() == [0]
