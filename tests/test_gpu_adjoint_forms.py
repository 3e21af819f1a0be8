"""Which form of d/dphi a list takes, and that both agree: the push form where
the cell columns' windows fit its accumulators, the transposed form where they
do not and the list has the map; a list without stored windows takes the
transposed form at any size."""
import numpy as np
import pytest

import oracle as O
from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MASK = vct.VCT_OUT_LAP | vct.VCT_OUT_PZ
CUBIC = I.KERNEL_CUBIC_SPLINE

SETS = {
    "3d": (lambda: I.small("sigma3d"), False),
    "3d-cubic": (lambda: I.make_sigma3d(20, 18, 11, 0.05, kernel=CUBIC), False),
    "3d-tall": (lambda: I.make_sigma3d(14, 13, 120, 0.05), True),   # column windows of 9 x 1,365 particles
    "2d": (lambda: I.small("bfe2d"), False),
    "2d-tall": (lambda: I.make_2d(40, 700, 1.0, 0.10), True),       # 3 x 2,154
}


def forms(w, u, g, win):
    g.nl.chunk_win = win
    vct.vct_timing_reset()
    vct.vct_timing_enable(True)
    try:
        dphi, _ = g.adjoint(u, want_dtheta=False)
        torch.cuda.synchronize()
    finally:
        vct.vct_timing_enable(False)
    names = set(vct.vct_timing_read())
    vct.vct_timing_reset()
    return g.unsort(dphi).cpu().numpy(), names


@pytest.mark.parametrize("name", list(SETS))
def test_forms(name):
    make, wide = SETS[name]
    w = make()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=True)
    g.moments(w.mapspec, MASK)
    uh = np.random.default_rng(3).standard_normal(w.n)
    u = g.sorted_field(uh)[0].contiguous()
    win, col_t = g.nl.chunk_win, g.nl.col_t
    auto, names = forms(w, u, g, win)
    assert ("k_adjoint_weights" in names) == wide and ("k_adjoint_push" in names) != wide
    trans, names = forms(w, u, g, None)
    assert "k_adjoint_weights" in names
    g.nl.col_t = None
    push, names = forms(w, u, g, win)
    assert "k_adjoint_push" in names and "k_adjoint_weights" not in names
    g.nl.col_t = col_t
    assert np.array_equal(auto, trans if wide else push)
    # both forms sum the same FP64 weights: 1e-13 of the largest (the bound the push form's resolution gives)
    sc = np.abs(trans).max()
    assert np.abs(push - trans).max() <= 1e-13 * sc
    ks = np.sort(np.random.default_rng(4).choice(w.n, 48, replace=False))
    ref = O.adjoint_dphi(w.pos, w.vol, w.kernel, w.R, w.mapspec, uh, ks=ks)
    assert np.abs(auto[ks] - ref).max() <= 1e-10 * np.abs(ref).max()
