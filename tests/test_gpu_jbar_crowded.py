"""Volume smoothing of a cell whose targets span more than four chunks in a block
that fits the LDS area (the windows of such a cell do not: its first wave takes
the targets one after the other), in every launch shape, against the oracle's
sequential update.  Bar as for the plain sets: 1e-12 of each particle's Jbar."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from test_gpu_jbar import CV, DEV, _check, _oracle_in_schedule_order, _sigma_J

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _crowded(dim, extra):
    w = I.make_2d(40, 30, 1.0, 0.10) if dim == 2 else \
        I.make_sigma3d(15, 14, 12, 0.05, kernel=I.KERNEL_CUBIC_SPLINE, nx_span=15)
    _, dims = vct.vct_grid_dims(dim, w.lo, w.hi, w.R)
    cell = [w.hi[a] / dims[a] for a in range(dim)]
    rng = np.random.default_rng(11)
    spot = np.stack([(dims[a] // 2 + rng.uniform(0.05, 0.95, extra)) * cell[a] for a in range(dim)])
    w.pos = np.ascontiguousarray(np.concatenate([w.pos, spot], axis=1))
    w.vol = np.concatenate([w.vol, np.full(extra, w.vol[0])])
    return w


def _largest(g):
    """(targets, block, chunks) of the largest cell."""
    cs, start = g.cell_start.cpu().numpy(), g.chunk_start.cpu().numpy()
    own = np.diff(cs).reshape(g.dims[: g.dim])
    pad = np.pad(own, 1)
    k = int(np.diff(cs).argmax())
    at = np.unravel_index(k, own.shape)
    block = int(pad[tuple(slice(c, c + 3) for c in at)].sum())
    first = np.searchsorted(start[: int(g.chunk_off[-1])], [cs[k], cs[k + 1] - 1], side="right") - 1
    return int(own[at]), block, int(first[1] - first[0]) + 1


@pytest.mark.parametrize("dim,extra", [(2, 300), (2, 700), (3, 300), (3, 440)])
def test_crowded_cell(dim, extra):
    w = _crowded(dim, extra)
    J = _sigma_J(w) if w.dim == 3 else 1.0 + 0.3 * np.random.default_rng(3).uniform(size=w.n)
    jb0 = J * I.volume_perturbation(w.n)
    ref = _oracle_in_schedule_order(w, J, jb0, CV)
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=False)
    targets, block, chunks = _largest(g)
    assert targets >= extra and block <= 1024 and chunks > 4, (targets, block, chunks)
    for nnz in (g.nnz, 0):
        g.nl.nnz = nnz
        jbs = g.sorted_field(jb0)[0].contiguous()
        g.jbar_smooth(g.sorted_field(J)[0].contiguous(), jbs, CV)
        _check(f"{dim}-D, {extra}", w, J, jb0, g.unsort(jbs[: g.n]).cpu().numpy(), ref)
    g.nl.nnz = g.nnz
