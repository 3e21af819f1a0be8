"""The moment sweeps' launch classes against the oracle: the state they feed,
through an FP64 apply, on short-row and long-row sets with rows beyond a
class's register slots and windows beyond its LDS capacity, each with the class
its mean row length selects and with nnz unset in the list (the long class)."""
import pytest

import oracle as O
from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from _parity import fp64_check, oracle_rows
from test_gpu_row_classes import MASK, SETS

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _wide():
    w = I.small("sigma3d")
    w.R *= 1.4
    return w


MORE = {name: make for name, (make, _, _) in SETS.items()}
MORE["3d"] = lambda: I.small("sigma3d")
MORE["3d-wide"] = _wide


@pytest.mark.parametrize("name", list(MORE))
def test_state_of_either_class(name):
    w = MORE[name]()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device="cuda:0", keep_col=False)
    phi = g.sorted_field(w.phi)
    rec, fl = O.sph2(w.pos, w.vol, w.phi, w.kernel, w.R, w.mapspec)
    assert not fl.any()
    ref = oracle_rows(rec, w.dim, MASK)
    for nnz in (g.nnz, 0):
        g.nl.nnz = nnz
        assert g.moments(w.mapspec, MASK) == vct.VCT_OK
        got = g.unsort(g.apply(phi, vct.VCT_FP64)[:, : g.n]).cpu().numpy()
        fp64_check(w, w.kernel, w.R, got, ref, MASK, label=f"{name}, nnz {nnz}")
    g.nl.nnz = g.nnz
