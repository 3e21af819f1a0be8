"""The transposed-entry map reports any entry whose transpose is not in its place
(VCT_E_HIP), wherever in a row it lies: the hit words of a search are changed
between its two calls so that one particle has a wrong neighbour, the number of
its neighbours and so every row's length unchanged."""
import ctypes as C

import numpy as np
import pytest

from paper_2607_28872_amd import inputs as I
from paper_2607_28872_amd import vct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def word_offset(n, ncell):
    """Where the hit words begin in the workspace (counts, scan tiles, the search's state)."""
    m, off = max(n, ncell), 0
    for size in (4 * m, 8 * ((m + 2047) // 2048), 24 + 256 * 8, 0):
        off = (off + 255) // 256 * 256 + size
    return off


@pytest.mark.parametrize("family", ["bf2d", "sigma3d"])
@pytest.mark.parametrize("offsets", [True, False])   # window offsets from col16, or from the columns
def test_every_entry_is_checked(family, offsets):
    w = I.small(family)
    g = vct.Geometry(w.pos, w.vol, w.lo, w.hi, w.R, w.kernel, device=DEV)
    nl = vct.vct_nlist.from_buffer_copy(g.nl)
    if not offsets:
        nl.col16 = None
    ws = g._nws
    start = g.chunk_start.cpu().numpy()
    chunks = int(g.chunk_off[-1])
    W = g.chunk_win.cpu().numpy()
    nr, off = W[:, 0], W[:, 20:30]   # ranges, (pad, 9 64-bit starts,) 10 offsets
    rng = np.random.default_rng(2)

    def rows():
        return vct.vct_neighbors_rows(nl, g.pos, g.nnz, 1, ws)

    assert vct.vct_neighbors_search(nl, g.pos, ws) == (g.nnz, 1)
    words = ws[word_offset(g.n, g.ncell):][: g.n * 64 * 4].view(torch.int32)
    assert rows() == vct.VCT_OK
    clean = g.col_t.clone()
    done = 0
    while done < 24:
        b = int(rng.integers(chunks))
        p0, np_ = int(start[b]), int(start[b + 1] - start[b])
        pl, wd = int(rng.integers(np_)), int(rng.integers((off[b, nr[b]] + 31) // 32))
        at = p0 * 64 + wd * np_ + pl
        bits = int(words[at]) & 0xFFFFFFFF
        size = min(32, int(off[b, nr[b]]) - 32 * wd)
        hits = [k for k in range(size) if bits >> k & 1]
        free = [k for k in range(size) if not bits >> k & 1]
        if not hits or not free:
            continue
        new = bits & ~(1 << rng.choice(hits)) | 1 << int(rng.choice(free))
        words[at] = new - (1 << 32) if new >> 31 else new
        with pytest.raises(vct.VctError):
            rows()
        done += 1
        assert vct.vct_neighbors_search(nl, g.pos, ws) == (g.nnz, 1)
    assert rows() == vct.VCT_OK
    assert torch.equal(g.col_t, clean)
