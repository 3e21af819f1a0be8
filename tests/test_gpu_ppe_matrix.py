"""The pressure system's matrix as the solver applies it against the operator:
with rhs = A p formed from vct_apply_ops' Laplacian row and the Dirichlet
values, the solver's residual of the start value p (no iterations) is rounding.
Both launch classes, masks whose Laplacian row stands at different places, rows
beyond the register slots and windows beyond the LDS capacity."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from test_gpu_row_classes import CUBIC, with_patch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SETS = {
    "2d": lambda: (I.make_2d(72, 56, 1.0, 0.10), 1.0),
    "2d-patch": lambda: (with_patch(I.make_2d(120, 100, 1.0, 0.10), 12), 1.0),
    "2d-long": lambda: (I.make_2d(60, 50, 1.0, 0.10), 1.6),
    "3d": lambda: (I.small("sigma3d"), 1.0),
    "3d-wide": lambda: (I.small("sigma3d"), 1.4),
    "3d-cubic-patch": lambda: (with_patch(I.make_sigma3d(52, 50, 14, 0.05, kernel=CUBIC), 5), 1.0),
}


@pytest.mark.parametrize("mask", [vct.VCT_OUT_LAP, vct.VCT_OUT_LAP | vct.VCT_OUT_PZ, vct.VCT_OUT_DEFAULT], ids=str)
@pytest.mark.parametrize("name", list(SETS))
def test_residual_of_the_operators_own_rhs(name, mask):
    w, Rs = SETS[name]()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, Rs * w.R, w.kernel, device=DEV, keep_col=False)
    assert g.moments(w.mapspec, mask) == vct.VCT_OK
    rng = np.random.default_rng(5)
    p = torch.as_tensor(rng.standard_normal(w.n), device=DEV)   # rough: the Laplacian's terms do not cancel
    fixed = torch.as_tensor((rng.random(w.n) < 0.2).astype(np.uint8), device=DEV)
    row = {vct.VCT_OUT_LAP: 0, vct.VCT_OUT_LAP | vct.VCT_OUT_PZ: 0, vct.VCT_OUT_DEFAULT: w.dim}[mask]
    lap = g.apply(p.reshape(1, -1), vct.VCT_FP64)[0, :, row]
    ws = torch.empty(vct.lib().vct_ppe_workspace_size(w.dim, w.n, mask), dtype=torch.uint8, device=DEV)
    for d in (fixed, None):
        rhs = torch.where(fixed.bool(), p, lap) if d is not None else lap.contiguous()
        x = p.clone()
        _, it, rr = vct.vct_ppe_solve(g.nl, g.pos, g.vol, g.kernel, g.state64, mask, d, rhs.contiguous(), x, 0.0, 0, ws)
        # two orders of the same sums of at most 465 FP64 terms
        assert it == 0 and rr <= 465 * 2.0 ** -53, (name, mask, rr)
        assert torch.equal(x, p)
