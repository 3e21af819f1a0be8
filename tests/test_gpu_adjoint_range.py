"""d/dphi of cotangents that range over many orders of magnitude inside a cell
column: every particle's sum is as accurate as FP64 sums of its own terms,
however large the others' are, in every form: transposed, push with records in
LDS, push in passes.  (Lists of more than 10,240 particles without the
transposed-entry map keep one word per sum: there the bar is relative to the
largest.)  The bar is per particle, against sums of weights formed
here in FP64 from the same state: 64 u of its own sum of |terms|, the terms of
a weight taken by magnitude and the kernel shape with its slope (a rounding of
|r| moves it by that): about 20 roundings form a weight, and a sum of up to 200
terms over 8 lanes takes 30 more."""
import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MASK = vct.VCT_OUT_LAP | vct.VCT_OUT_PZ
CUBIC = I.KERNEL_CUBIC_SPLINE



def _tower():
    """A lattice of 12 layers with a block of 6 x 6 x 100: few, wide columns."""
    w = I.make_sigma3d(48, 48, 12, 0.05)
    block = I.lattice((6, 6, 100), w.dx, 0.05, seed=5, shuffle=False, origin=[21 * w.dx, 21 * w.dx, 0.0])
    keep = ~np.all(np.abs(w.pos[:2] - 24 * w.dx) < 3 * w.dx, axis=0)
    w.pos = np.ascontiguousarray(np.concatenate([w.pos[:, keep], block], axis=1))
    w.vol = np.full(w.pos.shape[1], w.dx ** 3)
    w.hi = (w.hi[0], w.hi[1], 100 * w.dx)
    return w


def columns(g):
    """Window particles of every cell column."""
    nz = g.dims[g.dim - 1]
    own = np.diff(g.cell_start.cpu().numpy()[::nz]).reshape(g.dims[: g.dim - 1])
    own = np.pad(own, 1)
    if g.dim == 2:
        return own[:-2] + own[1:-1] + own[2:]
    rows = own[:-2] + own[1:-1] + own[2:]
    return rows[:, :-2] + rows[:, 1:-1] + rows[:, 2:]


SETS = {
    "3d-tower": _tower,
    "3d": lambda: I.small("sigma3d"),
    "3d-cubic": lambda: I.make_sigma3d(20, 18, 11, 0.05, kernel=CUBIC),
    "3d-tall": lambda: I.make_sigma3d(14, 13, 120, 0.05),   # column windows of 9 x 1,365 particles
    "3d-tall-small": lambda: I.make_sigma3d(9, 9, 120, 0.05),
    "2d-tall-small": lambda: I.make_2d(12, 800, 1.0, 0.10),
    "2d": lambda: I.small("bfe2d"),
    "2d-tall": lambda: I.make_2d(40, 700, 1.0, 0.10),       # 3 x 2,154
    "2d-between": lambda: I.make_2d(40, 380, 1.0, 0.10),    # 3 x 1,170: records and one word in LDS, not two
    "2d-between-small": lambda: I.make_2d(24, 380, 1.0, 0.10),
}


def cotangent(kind, w, rng):
    z = w.pos[-1] / w.hi[-1]
    u = rng.standard_normal(w.n)
    if kind == "normal":
        return u
    if kind.startswith("depth"):
        return u * 10.0 ** (-float(kind[5:]) * z)
    if kind == "gauss":
        return u * np.exp(-0.5 * ((w.pos - w.pos.mean(axis=1, keepdims=True)) / 0.03) ** 2).prod(axis=0)
    if kind == "random":
        return u * 10.0 ** rng.uniform(-40, 40, w.n)
    assert kind == "spikes"
    u[rng.choice(w.n, 5, replace=False)] *= 1e25
    u[rng.choice(w.n, w.n // 3, replace=False)] = 0.0
    return u


def sums(g, w, uh):
    """(dphi, sum of |terms|) of every sorted particle, from the state, in FP64."""
    d, n, nL, m = w.dim, g.n, (3 if w.dim == 2 else 6), (3 if w.dim == 2 else 6)
    nk = d + m
    pairs = [(0, 0), (1, 1), (0, 1)] if d == 2 else [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]
    state, pos, vol = (t.cpu().numpy() for t in (g.state64, g.pos[:, :n], g.vol[:n]))
    rp, col = g.row_ptr.cpu().numpy(), g.col[: g.nnz].cpu().numpy()
    i = np.repeat(np.arange(n), np.diff(rp))
    L, P = state[:nL, :n], state[nL: nL + nk, :n]   # the Laplacian row comes first in this mask
    r = (pos[:, col] - pos[:, i]) / w.R
    q = np.sqrt((r * r).sum(axis=0))
    if w.kernel == CUBIC:
        s = 2 * q
        c = np.where(s <= 1, 3 - 2.25 * s, 0.75 * (2 - s) ** 2 / s)
        slope = np.where(s <= 1, 4.5, 1.5 * (2 * (2 - s) / s + ((2 - s) / s) ** 2))
    else:
        c, slope = (1 - q) ** 3, 3 * (1 - q) ** 2
    qq = np.stack([r[a] * r[b] for a, b in pairs])
    two = np.array([1.0 if a == b else 2.0 for a, b in pairs])[:, None]
    V = vol[col]

    def weights(L, P, r, qq, c):
        rLr, sa, ss = (two * L[:, i] * qq).sum(axis=0), (P[:d, i] * r).sum(axis=0), (P[d:, i] * qq).sum(axis=0)
        return V * c * (sa + rLr * ss / q ** 4)

    out = []
    for wt, uu, sign in ((weights(L, P, r, qq, c), uh, -1.0),
                         (weights(abs(L), abs(P), abs(r), abs(qq), c + slope), abs(uh), 1.0)):
        t = (uu[i] * wt).astype(np.longdouble)
        a = np.zeros(n, np.longdouble)
        np.add.at(a, col, t)
        np.add.at(a, i, sign * t)
        out.append(a)
    return out


@pytest.mark.parametrize("name", list(SETS))
def test_each_particle_by_its_own_terms(name):
    w = SETS[name]()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV, keep_col=True)
    assert g.moments(w.mapspec, MASK) == vct.VCT_OK
    wide = columns(g) > 3200
    assert wide.any() == (name == "3d-tower" or "tall" in name or "between" in name), name
    perm = g.perm[: g.n].long().cpu().numpy()
    win, col_t, count = g.nl.chunk_win, g.nl.col_t, g.nl.wide_particles
    for kind in ("normal", "depth6", "depth12", "depth30", "gauss", "random", "spikes"):
        uh = cotangent(kind, w, np.random.default_rng(3))[perm]
        u = torch.as_tensor(uh, device=DEV)
        ref, mag = sums(g, w, uh)
        for form in ("auto", "transposed", "push", "passes"):   # (passes: wide columns in a list with the map)
            one_word = form == "push" and g.n > 10240
            if one_word and kind != "normal":
                continue
            g.nl.chunk_win = None if form == "transposed" else win
            g.nl.col_t = None if form == "push" else col_t
            if form == "passes" and not name.endswith("-small"):
                continue
            g.nl.wide_particles = 0 if form == "passes" else count   # (0: a small set then takes the push form)
            got = g.adjoint(u, want_dtheta=False)[0].cpu().numpy()
            err = np.abs(got - ref)
            if one_word:
                assert err.max() <= 1e-13 * np.abs(ref).max()
                continue
            bad = err > 64 * 2.0 ** -53 * mag + 2.0 ** -1000
            assert not bad.any(), (kind, form, int(bad.sum()), float((err / np.maximum(mag, 1e-290)).max()))
            assert np.array_equal(got, g.adjoint(u, want_dtheta=False)[0].cpu().numpy()), (kind, form)
