"""The neighbour search's matrix-core test against the definition, pair by pair
on the CPU: d2 summed left to right in FP64, d2 < R^2, no particle its own
neighbour.  The sets sit where the split into certain and re-tested candidates
can go wrong: distances exactly at R, coordinates far from the origin, scales
beyond FP32, positions far outside the box, few and odd numbers of particles
(idle columns of the products), and windows over one segment (1,536 records),
over the staging words (2,048) and over several segments.  The rows are compared
as they are: equal, entry by entry."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lattice(counts):
    dx = 1.0 / counts[0]
    return I.lattice(counts, dx, 0.0, seed=1, shuffle=True), [c * dx for c in counts], 3.0 * dx


def _cloud(n, dim, R, seed, size=1.0):
    return np.random.default_rng(seed).uniform(0.0, size, (dim, n)), [size] * dim, R


def _astray():
    pos, hi, R = _cloud(900, 3, 0.21, 4)
    pos[:, 50:54] = 1e35      # four at one place, far outside
    pos[0, 60:63] = [1e12, 1e12 + 0.125, 3.5]
    pos[1:, 60:63] = pos[1:, 60:61]
    return pos, hi, R


SETS = {
    "3d-ties": lambda: _lattice((13, 12, 11)),
    "2d-ties": lambda: _lattice((40, 33)),
    "astray": _astray,
    "one-segment": lambda: _cloud(2900, 3, 0.24, 5),         # windows of up to about 2,000
    "two-segments": lambda: _cloud(3600, 3, 0.3, 6),         # windows beyond the staging words
    "three-segments": lambda: _cloud(4100, 2, 0.45, 7),
}
for k in (1, 2, 15, 16, 17, 33, 64, 65):
    SETS[f"3d-{k}"] = lambda k=k: _cloud(k, 3, 0.3, 20 + k)
    SETS[f"2d-{k}"] = lambda k=k: _cloud(k, 2, 0.3, 40 + k)


def _rows(pos, R):
    with np.errstate(invalid="ignore", over="ignore"):
        d2 = np.square(pos[0][:, None] - pos[0][None, :])
        for a in range(1, pos.shape[0]):
            d2 = d2 + np.square(pos[a][:, None] - pos[a][None, :])
        near = d2 < R * R
    np.fill_diagonal(near, False)
    return near


@pytest.mark.parametrize("scale,shift", [(1.0, 0.0), (1e-25, 0.0), (1e25, 0.0), (1.0, 4096.0)])
@pytest.mark.parametrize("name", list(SETS))
def test_rows_are_the_definition(name, scale, shift):
    pos, hi, R = SETS[name]()
    pos = np.ascontiguousarray(pos * scale + shift)
    R = R * scale
    n, dim = pos.shape[1], pos.shape[0]
    lo, hi = [shift] * dim, [h * scale + shift for h in hi]
    vol = np.full(n, 1.0)
    g = vct.Geometry(pos, vol, lo, hi, R, I.KERNEL_WENDLAND_C2, device="cuda:0")
    perm = g.perm[:n].cpu().numpy().astype(np.int64)
    rp, col = g.row_ptr.cpu().numpy(), g.col.cpu().numpy()
    near = _rows(pos[:, perm], R)
    assert np.array_equal(np.diff(rp[: n + 1]), near.sum(axis=1))
    want = np.nonzero(near)
    assert np.array_equal(col[: rp[n]], want[1])
