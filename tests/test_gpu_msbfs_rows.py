"""Batched BFS at the row lengths where its expansion changes path (0 and 1,
the edges of a 64-edge step and of a 256-edge piece, several pieces), with
rows of both sides of a 16-vertex group, whole and partial query words, and
a session whose lanes are reused: levels against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENS = [0, 1, 2, 15, 16, 17, 63, 64, 65, 255, 256, 257, 512, 513, 1300]


@pytest.fixture(scope="module")
def grb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_01407_amd as g
    return g


@pytest.fixture(scope="module", params=[5000, 5041], ids=["n5000", "n5041"])
def rows(request):
    """A hub per length over its own targets, a path through the hubs, a few
    shared targets; ids at random."""
    n = request.param
    rng = np.random.default_rng(n)
    ids = rng.permutation(n)
    src, dst, at = [], [], len(LENS)
    for i, k in enumerate(LENS):
        leaves = ids[at: at + k]
        at += k
        src += [ids[i]] * k + list(leaves[::7])
        dst += list(leaves) + list(rng.choice(ids[len(LENS):at + 1], leaves[::7].size))
        src.append(ids[i])
        dst.append(ids[(i + 1) % len(LENS)])
    g = graphgen.from_edges("rows", n, np.array(src), np.array(dst))
    return g, oracle.Adjacency.from_raw(g), ids


@pytest.mark.parametrize("k", [1, 63, 65, 200])
@pytest.mark.parametrize("direction", [0, 1, 2], ids=["auto", "push", "pull"])
def test_rows(grb, rows, k, direction):
    g, adj, ids = rows
    src = ids[:k].astype(np.int32)
    ref = oracle.msbfs(adj, src, nthreads=8)
    A = grb.Matrix.from_raw(g)
    for kt in sorted({min(x, (k + 63) // 64) for x in (1, 2, 8)}):
        lev = grb.msbfs(A, src, words_per_pass=kt, desc=grb.descriptor(direction=direction))
        assert np.array_equal(lev.cpu().numpy().T, ref), kt


@pytest.mark.parametrize("direction", [1, 2], ids=["push", "pull"])
def test_reused_lanes(grb, rows, direction):
    g, adj, ids = rows
    ss = grb.MsbfsSession(grb.Matrix.from_raw(g), 70, desc=grb.descriptor(direction=direction))
    for turn in range(3):  # the lanes of both words again, from other sources
        lanes = [0, 5, 63, 64, 69]
        src = [int(v) for v in ids[5 * turn: 5 * turn + 5]]
        ss.join(lanes, src)
        left = set(lanes)
        for _ in range(100):
            done, _ = ss.step(3)
            left -= set(done)
            if not left:
                break
        out = ss.extract(lanes).cpu().numpy()
        for i, s in enumerate(src):
            assert np.array_equal(out[i], oracle.bfs(adj, s, parents=False)[0]), (turn, s)
