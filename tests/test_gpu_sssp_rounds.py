"""SSSP pull rounds at the row lengths where they change path (the edges of
a 256-entry piece, several pieces of one row in a wave's run and over two
runs), with distances that tie, zero and equal weights, rows settled below the
frontier, and weights whose sums round: distances in every direction mode
against the oracle, for the weights whose sums round against the least fixed
point of the float32 relaxation (the oracle adds in double)."""
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


def _hubs(n, lens, rng):
    """Hubs of the given degrees with shared leaves, a path through the hubs."""
    ids = rng.permutation(n)
    hubs, rest = ids[: len(lens)], ids[len(lens):]
    src = np.concatenate([np.full(k, h) for h, k in zip(hubs, lens)] + [hubs, rest[:-1:9]])
    dst = np.concatenate([rng.choice(rest, size=k, replace=False) for k in lens]
                         + [np.roll(hubs, 1), rest[1::9][: rest[:-1:9].size]])
    return src, dst, hubs


def _fixed_point(adj, s):
    rp, ci, w = adj.arrays(weights=True)[:3]
    row, w = np.repeat(np.arange(adj.n), np.diff(rp)), np.asarray(w, np.float32)
    d = np.full(adj.n, np.inf, np.float32)
    d[s] = 0
    while True:
        nxt = d.copy()
        np.minimum.at(nxt, ci, d[row] + w)
        if np.array_equal(nxt, d):
            return d
        d = nxt


@pytest.mark.parametrize("weights", ["whole", "zero_and_one", "equal", "fine"])
@pytest.mark.parametrize("direction", [0, 1, 2], ids=["auto", "push", "pull"])
def test_pull_rows(grb, weights, direction):
    rng = np.random.default_rng(8)
    n = 9001
    src, dst, hubs = _hubs(n, [1, 63, 64, 65, 255, 256, 257, 511, 513, 4000, 6000, 6001], rng)
    m = src.size
    w = {"whole": rng.integers(1, 65, m), "zero_and_one": rng.integers(0, 2, m),
         "equal": np.full(m, 3), "fine": rng.random(m) * 10.0 ** rng.integers(-6, 3, m)}[weights]
    g = graphgen.from_edges("hubs", n, src, dst, w.astype(np.float32))
    A = grb.Matrix.from_raw(g)
    adj = oracle.Adjacency.from_raw(g)
    for s in (int(hubs[0]), int(hubs[-1]), int(src[5000])):
        ref = _fixed_point(adj, s)
        if weights != "fine":
            assert np.array_equal(ref, oracle.sssp(adj, s)[0])
        got = grb.sssp(A, s, desc=grb.descriptor(direction=direction)).cpu().numpy()
        assert np.array_equal(got, ref), (s, weights)
