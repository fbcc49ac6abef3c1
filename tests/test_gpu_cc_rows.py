"""Connected components at the row lengths where its sweep changes path
(0 to 3 entries, the edges of a 256-entry piece, several pieces), in
components that hold the smallest id and in ones that do not, symmetric and
directed: labels against the oracle, iterations and change counts against a
numpy FastSV of the same steps."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def grb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_01407_amd as g
    return g


def _stars(lens, n, low, rng):
    """Hubs of the given degrees over disjoint leaves, some leaves linked to a
    leaf of the next star; `low` puts a separate pair at ids 0 and 1."""
    ids = rng.permutation(np.arange(2, n))
    src, dst, at, prev = [], [], 0, None
    for k in lens:
        hub, leaves = ids[at], ids[at + 1: at + 1 + k]
        at += 1 + k
        src += [hub] * k
        dst += list(leaves)
        if prev is not None and k % 2:
            src.append(prev)
            dst.append(leaves[0] if k else hub)
        prev = leaves[-1] if k else hub
    if low:
        src.append(0)
        dst.append(1)
    return np.array(src), np.array(dst)


def _fastsv(n, src, dst):
    """Iterations and change counts of FastSV with numpy (both directions)."""
    s, d = np.concatenate([src, dst]), np.concatenate([dst, src])
    keep = s != d
    s, d = s[keep], d[keep]
    f, f_old, gf, m = (np.arange(n) for _ in range(4))
    f, gf, m = f.copy(), gf.copy(), m.copy()
    changes = []
    while True:
        np.minimum.at(m, s, gf[d])
        np.minimum.at(f, f_old, m)
        f = np.minimum(np.minimum(f, m), gf)
        g = f[f]
        changes.append(int((g != gf).sum()))
        gf, f_old = g, f.copy()
        if changes[-1] == 0:
            return gf, changes


@pytest.mark.parametrize("low", [False, True], ids=["hub_low", "pair_low"])
@pytest.mark.parametrize("symmetric", [True, False], ids=["sym", "dir"])
@pytest.mark.parametrize("n", [4095, 4097, 70001])
def test_cc_row_lengths(grb, n, symmetric, low):
    rng = np.random.default_rng(n + low)
    src, dst = _stars([1, 2, 3, 64, 255, 256, 257, 511, 513, 1300], n, low, rng)
    g = graphgen.from_edges("stars", n, src, dst, None, symmetric)
    A = grb.Matrix.from_raw(g, weights=False)
    ref, _ = oracle.cc(oracle.Adjacency(n, g.src, g.dst, symmetrise=True))
    lab, it = grb.cc(A)
    assert np.array_equal(lab.cpu().numpy(), ref)
    want, changes = _fastsv(n, src, dst)
    assert np.array_equal(want, ref)
    assert it == len(changes)
    assert grb.last_stats()["frontier"] == changes
