"""The applies' launch classes (short and long rows) against the oracle.

The class follows the mean row length, so the sets here are short on average:
plain lattices of both kernels, and lattices with a patch of half the spacing,
whose rows exceed the class's register slots and whose windows exceed its LDS
capacity.  Each set also runs with nnz unset in the list, which selects the
long-row class on the same lists."""
import numpy as np
import pytest

import oracle as O
from oracle import extended as OX
from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

from _parity import fp64_check, oracle_rows, per_particle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
CUBIC = I.KERNEL_CUBIC_SPLINE
MASK = vct.VCT_OUT_DEFAULT | vct.VCT_OUT_PZ


def with_patch(w, cells):
    """w with the lattice sites of a central box of `cells` spacings a side
    replaced by 2^dim finer ones (half the spacing, the volumes to match)."""
    mid = [w.dx * (c // 2) for c in w.counts]
    half = 0.5 * cells * w.dx
    keep = ~np.all([np.abs(w.pos[a] - mid[a]) < half for a in range(w.dim)], axis=0)
    fine = I.lattice((2 * cells,) * w.dim, 0.5 * w.dx, w.jitter, seed=5, shuffle=False,
                     origin=[m - half for m in mid])
    w.pos = np.ascontiguousarray(np.concatenate([w.pos[:, keep], fine], axis=1))
    w.vol = np.concatenate([w.vol[keep], np.full(fine.shape[1], (0.5 * w.dx) ** w.dim)])
    quad = [I.random_quadratic(w.dim, 31), I.random_quadratic(w.dim, 32)]
    w.phi = np.stack([np.sin(3.0 * w.pos[0]) + I.eval_quadratic(quad[0], w.pos), I.eval_quadratic(quad[1], w.pos)])
    return w


SETS = {
    "2d": (lambda: I.make_2d(72, 56, 1.0, 0.10), 28, 448),
    "2d-cubic": (lambda: I.make_2d(72, 56, 1.0, 0.10, kernel=CUBIC), 28, 448),
    "3d-cubic": (lambda: I.make_sigma3d(30, 28, 12, 0.05, kernel=CUBIC), 64, 1184),
    "2d-patch": (lambda: with_patch(I.make_2d(120, 100, 1.0, 0.10), 12), 28, 448),
    "3d-cubic-patch": (lambda: with_patch(I.make_sigma3d(52, 50, 14, 0.05, kernel=CUBIC), 5), 64, 1184),
}


@pytest.mark.parametrize("name", list(SETS))
def test_row_classes(name):
    make, slots, win = SETS[name]
    w = make()
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV)
    assert g.nl.nnz // w.n <= (30 if w.dim == 2 else 62)   # the short class runs
    tab = g.chunk_win.cpu().numpy()
    nch = int(g.chunk_off[-1].item())
    widest = int(tab[np.arange(nch), 20 + tab[:nch, 0]].max())
    longest = int(np.diff(g.row_ptr.cpu().numpy()).max())
    print(f"\n{name}: longest row {longest} ({slots} slots), widest window {widest} ({win} records)")
    if "patch" in name:
        assert longest > slots and widest > win   # the tail loop and the memory path run
    g.moments(w.mapspec, MASK, fp32_copy=True)
    phi = g.sorted_field(w.phi)
    rec, fl = O.sph2(w.pos, w.vol, w.phi, w.kernel, w.R, w.mapspec)
    assert not fl.any()
    ref = oracle_rows(rec, w.dim, MASK)
    scale = np.abs(ref).max(axis=1, keepdims=True)
    kap = OX.moment_condition(w.pos, w.vol, w.kernel, w.R, rows=np.arange(w.n))
    ng = w.dim
    mixed = []
    for nnz in (g.nnz, 0):
        g.nl.nnz = nnz
        got = {p: g.unsort(g.apply(phi, p)[:, : g.n]).cpu().numpy()
               for p in (vct.VCT_FP64, vct.VCT_MIXED, vct.VCT_MIXED_S64)}
        fp64_check(w, w.kernel, w.R, got[vct.VCT_FP64], ref, MASK, label=f"{name}, nnz {nnz}")
        # FP32 sums of up to 16 terms a lane and two combining steps (20 u of
        # the terms' magnitude, u = 2^-24), amplified by at most kappa; the
        # bars of well-conditioned particles are those of the mixed form
        for p in (vct.VCT_MIXED, vct.VCT_MIXED_S64):
            for rows, bar in ((slice(0, ng), 1e-5), (slice(ng, None), 1e-4)):
                e = per_particle(got[p][..., rows], ref[..., rows], scale[..., rows])
                assert np.all(e <= np.maximum(bar, 20 * 2.0 ** -24 * kap)), (name, nnz, p, e.max())
        mixed.append((got[vct.VCT_MIXED], got[vct.VCT_MIXED_S64]))
    g.nl.nnz = g.nnz
    # the mixed form sums in the same order in both classes
    assert np.array_equal(mixed[0][0], mixed[1][0]) and np.array_equal(mixed[0][1], mixed[1][1])
