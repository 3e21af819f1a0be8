"""d/dphi does not depend on the units: lengths and volumes scaled by powers of
two scale every weight by an exact power of two (the identity map), as long as
the weights, the moments and the state are in range.  The push form's bound on
its terms has to stay in range with them."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MASK = vct.VCT_OUT_LAP | vct.VCT_OUT_PZ


def dphi(w, length, volume, push):
    g = vct.Geometry(w.pos * length, w.vol * volume, w.lo, tuple(h * length for h in w.hi), w.R * length, w.kernel,
                     device=DEV, keep_col=not push)
    assert g.moments(I.MapSpec(kind=I.MAP_IDENTITY), MASK) == vct.VCT_OK
    if not push:
        g.nl.chunk_win = None
    u = g.sorted_field(np.random.default_rng(3).standard_normal(w.n))[0].contiguous()
    return g.unsort(g.adjoint(u, want_dtheta=False)[0]).cpu().numpy()


@pytest.mark.parametrize("family", ["bf2d", "sigma3d"])
@pytest.mark.parametrize("length,volume", [(-200, -130), (-230, -70), (200, 130), (3, -5)])
def test_scaled_units(family, length, volume):
    w = I.small(family)
    for push in (True, False):
        ref = dphi(w, 1.0, 1.0, push)
        got = dphi(w, 2.0 ** length, 2.0 ** volume, push) * 4.0 ** length
        # exact but for the volumes' share of sums that lose nothing: 1e-12 of the largest
        assert np.isfinite(got).all(), (family, push)
        assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max(), (family, push)
