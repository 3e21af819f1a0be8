"""The form of d/dphi that a list with the transposed-entry map takes: by the
particles of wide cell columns (whatever part of the box is empty), by the
length of the rows and by the number of entries; and the count the search
leaves of the particles in wide columns."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from test_gpu_adjoint_range import _tower, columns

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MASK = vct.VCT_OUT_LAP | vct.VCT_OUT_PZ


def _box(w, *times):
    w.hi = tuple(h * t for h, t in zip(w.hi, times))
    return w



SETS = {   # transposed?
    "2d-tall": (lambda: I.make_2d(40, 1200, 1.0, 0.10), True),
    "2d-tall-half-box": (lambda: _box(I.make_2d(40, 1200, 1.0, 0.10), 2, 1), True),
    "3d-tall-empty-box": (lambda: _box(I.make_sigma3d(14, 13, 120, 0.05), 3, 3, 1), True),
    "3d-tower": (_tower, True),
    "2d-plain": (lambda: I.make_2d(300, 200, 1.0, 0.10), True),
    "3d-short-rows": (lambda: I.make_sigma3d(64, 64, 30, 0.05, kernel=I.KERNEL_CUBIC_SPLINE), False),
    "3d-long-rows": (lambda: I.make_sigma3d(52, 52, 30, 0.05), False),
    "3d-small": (lambda: I.small("sigma3d"), False),
}


def particles_in_wide(g):
    nz = g.dims[g.dim - 1]
    own = np.diff(g.cell_start.cpu().numpy()[::nz]).reshape(g.dims[: g.dim - 1])
    return int(own[columns(g) > 3200].sum())


@pytest.mark.parametrize("name", list(SETS))
def test_choice(name):
    make, transposed = SETS[name]
    w = make()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=True)
    g.moments(w.mapspec, MASK)
    u = torch.ones(g.n, dtype=torch.float64, device=DEV)
    vct.vct_timing_reset()
    vct.vct_timing_enable(True)
    try:
        g.adjoint(u, want_dtheta=False)
        torch.cuda.synchronize()
    finally:
        vct.vct_timing_enable(False)
    names = set(vct.vct_timing_read())
    vct.vct_timing_reset()
    print(name, g.n, g.nnz, sorted(names))
    assert ("k_adjoint_weights" in names) == transposed and ("k_adjoint_push" in names) != transposed
    assert g.nl.wide_particles == 1 + particles_in_wide(g)
    assert ("k_adjoint_push (wide)" in names) == (not transposed and g.nl.wide_particles > 1)


@pytest.mark.parametrize("name", ["3d-small", "3d-long-rows", "2d-plain", "2d-tall"])
def test_workspace_of_the_form(name):
    """The push form needs no room for the entries, the transposed form does."""
    make, transposed = SETS[name]
    w = make()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=True)
    g.moments(w.mapspec, MASK)
    u = torch.ones(g.n, dtype=torch.float64, device=DEV)
    want = g.adjoint(u, want_dtheta=False)[0]
    sizes = [vct.lib().vct_adjoint_workspace_size(g.dim, g.n, k, g.cmap.nterms) for k in (0, g.nnz)]
    for size, enough in ((sizes[0] - 1, False), (sizes[0], not transposed), (sizes[1] - 1, not transposed),
                         (sizes[1], True)):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        dphi = torch.empty(g.n, dtype=torch.float64, device=DEV)
        args = (g.nl, g.pos, g.vol, g.kernel, g.state64, MASK, g.cmap, None, u, dphi, None, ws)
        if enough:
            vct.vct_apply_ops_adjoint(*args)
            assert torch.equal(dphi, want)
        else:
            with pytest.raises(vct.VctError):
                vct.vct_apply_ops_adjoint(*args)


@pytest.mark.parametrize("keep_col", [True, False])
def test_wrong_count_of_wide_columns_shows(keep_col):
    """A list that claims to have no wide column, and has: NaN there, not a sum left out."""
    w = I.make_2d(12, 800, 1.0, 0.10)
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=keep_col)
    g.moments(w.mapspec, MASK)
    assert (columns(g) > 3200).all() and g.nl.wide_particles == 1 + g.n
    g.nl.wide_particles = 1
    assert torch.isnan(g.adjoint(torch.ones(g.n, dtype=torch.float64, device=DEV), want_dtheta=False)[0]).all()
