"""Volume smoothing of particles that (nearly) coincide: distances down to where
their squares are subnormal or zero exchange as the sequential update does.
Bar as for the plain sets: 1e-12 of each particle's Jbar."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from test_gpu_jbar import CV, DEV, _check, _oracle_in_schedule_order, _sigma_J

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GAPS = (0.0, 1e-200, 3e-162, 1e-160, 1e-157, 2e-154, 1e-150, 1e-100, 1e-20)


@pytest.mark.parametrize("family", ["bf2d", "sigma3d", "cubic"])
def test_close_particles(family):
    w = I.make_sigma3d(21, 20, 17, 0.05, kernel=I.KERNEL_CUBIC_SPLINE, nx_span=21) if family == "cubic" else I.small(family)
    # a group at the corner of the box, where coordinates resolve any gap
    w.pos[:, : len(GAPS) + 1] = 0.0
    w.pos[0, 1: len(GAPS) + 1] = GAPS
    J = _sigma_J(w) if w.dim == 3 else 1.0 + 0.3 * np.random.default_rng(3).uniform(size=w.n)
    jb0 = J * I.volume_perturbation(w.n)
    ref = _oracle_in_schedule_order(w, J, jb0, CV)
    assert np.isfinite(ref).all()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=False)
    for nnz in (g.nnz, 0):
        g.nl.nnz = nnz
        jbs = g.sorted_field(jb0)[0].contiguous()
        g.jbar_smooth(g.sorted_field(J)[0].contiguous(), jbs, CV)
        _check(family, w, J, jb0, g.unsort(jbs[: g.n]).cpu().numpy(), ref)
    g.nl.nnz = g.nnz
