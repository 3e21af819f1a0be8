"""The pressure solver with its matrix kept in the workspace against the same
solver that forms it in every product (a workspace without room for it): one
iteration from zero gives the same iterate and residual up to the rounding of
two orders of the same FP64 sums.  Both launch classes, rows beyond the register
slots, windows beyond the LDS capacity, Dirichlet rows, and lists with more
entries than the workspace has room for, which keep the product form."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from test_gpu_row_classes import CUBIC, with_patch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MASK = vct.VCT_OUT_LAP
SETS = {   # kept: the entries fit
    "2d": (lambda: (I.make_2d(72, 56, 1.0, 0.10), 1.0), True),
    "2d-patch": (lambda: (with_patch(I.make_2d(120, 100, 1.0, 0.10), 12), 1.0), True),
    "2d-slots": (lambda: (I.make_2d(60, 50, 1.0, 0.10), 1.2), True),
    "2d-beyond": (lambda: (I.make_2d(60, 50, 1.0, 0.10), 1.6), False),
    "3d": (lambda: (I.small("sigma3d"), 1.0), True),
    "3d-slots": (lambda: (I.small("sigma3d"), 1.05), True),
    "3d-beyond": (lambda: (I.small("sigma3d"), 1.6), False),
    "3d-cubic-patch": (lambda: (with_patch(I.make_sigma3d(52, 50, 14, 0.05, kernel=CUBIC), 5), 1.0), True),
}


@pytest.mark.parametrize("name", list(SETS))
def test_kept_matrix_is_the_operator(name):
    make, kept = SETS[name]
    w, Rs = make()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, Rs * w.R, w.kernel, device=DEV, keep_col=False)
    assert g.moments(w.mapspec, MASK) == vct.VCT_OK
    rng = np.random.default_rng(6)
    rhs = torch.as_tensor(rng.standard_normal(w.n), device=DEV)
    fixed = torch.as_tensor((rng.random(w.n) < 0.2).astype(np.uint8), device=DEV)
    full = vct.lib().vct_ppe_workspace_size(w.dim, w.n, MASK)
    for nnz in (g.nnz, 0):
        g.nl.nnz = nnz
        got = []
        for size in (full, full - 1):
            ws = torch.empty(size, dtype=torch.uint8, device=DEV)
            x = torch.zeros(w.n, dtype=torch.float64, device=DEV)
            vct.vct_timing_reset()
            vct.vct_timing_enable(True)
            _, it, rr = vct.vct_ppe_solve(g.nl, g.pos, g.vol, g.kernel, g.state64, MASK, fixed, rhs, x, 0.0, 1, ws)
            vct.vct_timing_enable(False)
            ran = vct.vct_timing_read()
            vct.vct_timing_reset()
            assert it == 1 and ("k_ppe_matvec" in ran) == (kept and size == full), (name, size)
            got.append((x.cpu().numpy(), rr))
        (x0, r0), (x1, r1) = got
        # rows of under 500 terms, a handful of scalars from sums over the set:
        # rounding of 500 u, amplified by the iteration's ratios (bar 1e4)
        bar = 500 * 2.0 ** -53 * 1e4
        assert np.abs(x0 - x1).max() <= bar * np.abs(x1).max(), name
        assert abs(r0 - r1) <= bar * r1, name
    g.nl.nnz = g.nnz
