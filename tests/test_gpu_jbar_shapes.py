"""Volume smoothing in its launch shapes against the oracle's sequential update
in the same order: short rows (cubic spline, one wave per cell) and long rows
(the waves of a group taking turns), rows of more than 128 entries, blocks on
both sides of the size whose positions are staged, columns of more chunks than
a wave has lanes, and the long shape on short rows (nnz unset in the list).
Bar as for the plain sets: 1e-12 of each particle's Jbar."""
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from test_gpu_jbar import CV, DEV, _check, _oracle_in_schedule_order, _sigma_J

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import numpy as np


def _plane(R):
    w = I.small("bf2d")
    w.R = R * w.dx
    return w


def _wide():   # rows of about 137, blocks of 729 .. 1,000
    w = I.make_sigma3d(23, 23, 23, 0.05, name="wide", nx_span=23)
    w.R = 3.2 * w.dx
    return w


SETS = {
    "3d-cubic": lambda: I.make_sigma3d(21, 20, 17, 0.05, kernel=I.KERNEL_CUBIC_SPLINE, name="cubic", nx_span=21),
    "3d-wide": _wide,
    "3d-tall": lambda: I.make_sigma3d(7, 6, 440, 0.05, name="tall", nx_span=7),
    "3d-one-cell": lambda: I.make_sigma3d(3, 3, 4, 0.05, name="one", nx_span=3),
    "2d-long-rows": lambda: _plane(6.6),
}


@pytest.mark.parametrize("name", list(SETS))
def test_against_the_sequential_update(name):
    w = SETS[name]()
    J = _sigma_J(w) if w.dim == 3 else 1.0 + 0.3 * np.random.default_rng(3).uniform(size=w.n)
    jb0 = J * I.volume_perturbation(w.n)
    ref = _oracle_in_schedule_order(w, J, jb0, CV)
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=False)
    for nnz in (g.nnz, 0):
        g.nl.nnz = nnz
        jbs = g.sorted_field(jb0)[0].contiguous()
        g.jbar_smooth(g.sorted_field(J)[0].contiguous(), jbs, CV)
        _check(name, w, J, jb0, g.unsort(jbs[: g.n]).cpu().numpy(), ref)
    g.nl.nnz = g.nnz
