"""Structure-only products where the kernel changes path: rows of B from the
concatenated stream to units of 128 entries (31, 32, 33), units' ends (64,
127, 128, 129, 256, 257), more than 64 units in a batch of mask entries, mask
rows from whole to shared between groups (31, 32, 33) and over 64 entries,
columns around the ends of both bitmaps (32,768 and 65,536), tails of 127 to
300 entries; more rows than one pass of the grid has: every entry and the
count against the oracle."""
import numpy as np
import pytest

from oracle import mxm as omxm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGE = 32768  # columns of the bitmap


@pytest.fixture(scope="module")
def grb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_01407_amd as g
    return g


def _csr(rows):
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return rp, np.concatenate(rows).astype(np.int32)


def _rows(rng, lens, ncols, forced=()):
    out = []
    for k in lens:
        c = rng.choice(ncols, size=min(k, ncols), replace=False)
        out.append(np.unique(np.concatenate([c, np.array(forced, np.int64)])))
    return out


@pytest.mark.parametrize("ncols", [700, EDGE, EDGE + 1, 2 * EDGE, 2 * EDGE + 1, 70000])
def test_row_lengths(grb, ncols):
    rng = np.random.default_rng(ncols)
    blen = [0, 1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 600] * 12
    alen = [0, 1, 5, 63, 64, 65, 127, 128, 129, 300, 640] * 9
    forced = [c for c in (0, 31, 32, EDGE - 1, EDGE, 2 * EDGE - 1, 2 * EDGE) if c < ncols]
    B = _rows(rng, blen, ncols, forced)
    B[0] = B[0][:0]
    A = _rows(rng, alen, ncols, forced)
    A[3] = A[3][:0]
    # tails of the lengths around their LDS list's end
    A += [np.concatenate([[7], np.arange(ncols - k, ncols)]) for k in (1, 127, 128, 129, 300)]
    mlen = [0, 1, 31, 32, 33, 63, 64, 65, 128, 192]
    M = _rows(rng, [mlen[i % len(mlen)] for i in range(len(A))], len(B))
    shape = (len(A), len(B), ncols)
    (mrp, mci), (arp, aci), (brp, bci) = _csr(M), _csr(A), _csr(B)
    got = grb.mxm_masked(grb.Matrix(shape[0], shape[1], mrp, mci, None),
                         grb.Matrix(shape[0], ncols, arp, aci, None),
                         grb.Matrix(shape[1], ncols, brp, bci, None), "plus_pair_int32")
    ref = omxm.mxm_masked((shape[0], shape[1], mrp, mci, None), (shape[0], ncols, arp, aci, None),
                          (shape[1], ncols, brp, bci, None), "plus_pair_int32")
    assert np.array_equal(got.cpu().numpy(), ref)


def test_count_equals_entries(grb):
    """A lower triangle of 40,000 rows (several per wave), some of them long."""
    rng = np.random.default_rng(5)
    n = 40000
    rows = []
    for i in range(n):
        k = 300 if i % 97 == 0 else (40 if i % 11 == 0 else i % 5)
        rows.append(np.unique(rng.integers(0, max(1, min(i, 900)), size=k)) if i else
                    np.zeros(0, np.int64))
    rows = [r[r < i] for i, r in enumerate(rows)]
    rp, ci = _csr(rows)
    L = grb.Matrix(n, n, rp, ci, None)
    ref = omxm.mxm_masked(*[(n, n, rp, ci, None)] * 3, "plus_pair_int32")
    assert np.array_equal(grb.mxm_masked(L, L, L).cpu().numpy(), ref)
    assert grb.tricount(L) == int(ref.sum())
