"""The pressure solver over the ends of its batches of eight iterations: a limit
of iterations is met exactly and the residual reported is that of the iterate
returned; a solve that converges gives the same bits, iterations and status for
every limit beyond it, wherever in a batch it ends."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MASK = vct.VCT_OUT_LAP


@pytest.fixture(scope="module")
def problem():
    w = I.small("sigma3d")
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=False)
    assert g.moments(w.mapspec, MASK) == vct.VCT_OK
    fixed = g.sorted_field(I.boundary_layer(w.pos, w.lo, w.hi, w.R).astype(np.float64))[0, : w.n] > 0.5
    rhs = g.sorted_field(np.sin(7.0 * w.pos[0]) * np.cos(5.0 * w.pos[2]))[0, : w.n].contiguous()
    ws = torch.empty(vct.lib().vct_ppe_workspace_size(w.dim, w.n, MASK), dtype=torch.uint8, device=DEV)
    return w, g, fixed.to(torch.uint8).contiguous(), rhs, ws


def _solve(problem, tol, limit, x=None):
    w, g, fixed, rhs, ws = problem
    x = torch.zeros(w.n, dtype=torch.float64, device=DEV) if x is None else x.clone()
    return vct.vct_ppe_solve(g.nl, g.pos, g.vol, g.kernel, g.state64, MASK, fixed, rhs, x, tol, limit, ws) + (x,)


@pytest.mark.parametrize("limit", [0, 1, 2, 7, 8, 9, 16, 17])
def test_limit_of_iterations(problem, limit):
    st, it, rr, x = _solve(problem, 0.0, limit)
    assert st == vct.VCT_W_NOCONV and it == limit
    _, it0, rr0, x0 = _solve(problem, 0.0, 0, x)
    assert it0 == 0 and torch.equal(x0, x)
    # the same residual with the coefficients formed in the product: two orders
    # of the same sums, their rounding bounded by that of a vector of norm 1
    assert abs(rr - rr0) <= 1e-9 * max(rr0, 1e-3), (rr, rr0)


def test_converged_solves_do_not_depend_on_the_limit(problem):
    for tol in (1e-1, 1e-2, 1e-3, 1e-4):
        st, it, rr, x = _solve(problem, tol, 400)
        assert st == vct.VCT_OK and it < 400
        for limit in (it, it + 1, it + 8):
            st1, it1, rr1, x1 = _solve(problem, tol, limit)
            assert (st1, it1, rr1) == (st, it, rr) and torch.equal(x1, x), (tol, limit)
        st1, it1, _, _ = _solve(problem, tol, it - 1)
        assert st1 == vct.VCT_W_NOCONV and it1 == it - 1
