"""The one-sweep kernels in both launch classes (short and long rows): the
conventional operators, the summation gradient, the pressure right-hand side
and the corrector against the oracle, on sets with rows beyond a class's
register slots and windows beyond its LDS capacity, and with nnz unset in the
list (the long-row class on the same lists).  Bars as for the plain sets: 1e-12
of the row maximum for the conventional operators, 1e-11 for the pressure
step."""
import numpy as np
import pytest

import oracle as O
from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from _parity import normwise, oracle_rows
from test_gpu_ppe import DT, GAMMA, RHO, _dev, _fields, _host
from test_gpu_row_classes import SETS

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MASK = vct.VCT_OUT_LAP
ALL = vct.VCT_OUT_DEFAULT | vct.VCT_OUT_HESS | vct.VCT_OUT_PHESS


def wide3d():   # windows beyond the long class's window
    w = I.small("sigma3d")
    w.R *= 1.4
    return w


MORE = {name: make for name, (make, _, _) in SETS.items()}
MORE["3d"] = lambda: I.small("sigma3d")
MORE["3d-wide"] = wide3d


@pytest.mark.parametrize("name", list(MORE))
def test_against_the_oracle(name):
    w = MORE[name]()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=False)
    assert g.moments(w.mapspec, MASK) == vct.VCT_OK
    csr = O.neighbors(w.pos, w.R)
    rec, fl = O.ops0(w.pos, w.vol, w.phi, w.kernel, w.R, w.mapspec, csr=csr)
    assert not fl.any()
    ref0 = oracle_rows(rec, w.dim, ALL)
    rng = np.random.default_rng(8)
    rho = rng.uniform(0.9, 1.1, w.n)
    phys, proj, fl = O.grad_sum(w.pos, w.vol, w.phi[0], w.kernel, w.R, w.mapspec, rho=rho, csr=csr)
    assert not fl.any()
    ax = [0, 1, 2] if w.dim == 3 else [0, 2]
    refg = np.concatenate([phys[:, ax], proj[:, ax]], axis=1)
    v, jr, dirichlet, pbc = _fields(w)
    refp = O.ppe_rhs(w.pos, w.vol, w.kernel, w.R, w.mapspec, v, RHO, DT, GAMMA, jr=jr, dirichlet=dirichlet, pbc=pbc,
                     csr=csr)
    p = rng.uniform(-1, 1, w.n) + w.pos[0]
    refc = O.ppe_correct(w.pos, w.vol, w.kernel, w.R, w.mapspec, p, v, RHO, DT, csr=csr) - v
    vs = _dev(g, v)
    for nnz in (g.nnz, 0):
        g.nl.nnz = nnz
        got = g.unsort(g.apply0(w.mapspec, g.sorted_field(w.phi), ALL)[:, : g.n]).cpu().numpy()
        assert normwise(got, ref0).max() <= 1e-12, (name, nnz)
        got = g.unsort(g.grad_sum(w.mapspec, g.sorted_field(w.phi[0])[0], g.sorted_field(rho)[0])[: g.n]).cpu().numpy()
        assert np.all(np.abs(got - refg).max(0) <= 1e-12 * np.abs(refg).max(0)), (name, nnz)
        out = [torch.empty(g.n, dtype=torch.float64, device=DEV) for _ in range(3)]
        vct.vct_ppe_rhs(g.nl, g.pos, g.vol, g.kernel, g.state64, MASK, g.cmap, vs, RHO, DT, GAMMA, _dev(g, jr),
                        _dev(g, dirichlet), _dev(g, pbc), *out)
        for a, b in zip(out, refp):
            assert np.abs(_host(g, a) - b).max() <= 1e-11 * np.abs(b).max(), (name, nnz)
        vout = torch.empty_like(vs)
        vct.vct_ppe_correct(g.nl, g.pos, g.vol, g.kernel, g.state64, MASK, g.cmap, _dev(g, p), vs, RHO, DT, vout)
        assert np.abs(_host(g, vout) - v - refc).max() <= 1e-11 * np.abs(refc).max(), (name, nnz)
    g.nl.nnz = g.nnz
