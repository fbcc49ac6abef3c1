"""Batched BFS whose levels change between the one-kernel and the two-kernel form:
searches that start on a path (tiny frontiers), cross a random graph (every
vertex over several edges) and end on another path, with and without rows longer
than 64 entries; few and many queries, forced directions, level caps, and
sessions whose queries join before and after a change: levels against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CORE, TAIL = 20000, 45


@pytest.fixture(scope="module")
def grb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_01407_amd as g
    return g


@pytest.fixture(scope="module", params=["low", "hub"])
def tails(request):
    rng = np.random.default_rng(11)
    n = CORE + 4 * TAIL + 101
    s, d = [rng.integers(0, CORE, 5 * CORE)], [rng.integers(0, CORE, 5 * CORE)]
    ends = []
    for i in range(4):  # paths that leave the core
        path = np.concatenate([[i], np.arange(CORE + i * TAIL, CORE + (i + 1) * TAIL)])
        s.append(path[:-1])
        d.append(path[1:])
        ends.append(path[-1])
    hub = n - 101
    k = 100 if request.param == "hub" else 20
    s.append(np.full(k + 1, hub))
    d.append(np.concatenate([np.arange(n - 100, n - 100 + k), [5]]))
    p = rng.permutation(n)
    g = graphgen.from_edges("tails", n, p[np.concatenate(s)], p[np.concatenate(d)])
    return g, oracle.Adjacency.from_raw(g), p, p[np.array(ends)]


def _sources(p, ends, k, seed):
    rng = np.random.default_rng(seed)
    src = np.concatenate([np.resize(ends, k - k // 8), p[rng.integers(0, CORE, k // 8)]])
    return src.astype(np.int32)


@pytest.mark.parametrize("k", [3, 130, 700])
@pytest.mark.parametrize("direction", [0, 1, 2], ids=["auto", "push", "pull"])
def test_forms(grb, tails, k, direction):
    g, adj, p, ends = tails
    src = _sources(p, ends, k, k)
    ref = oracle.msbfs(adj, src, nthreads=8)
    A = grb.Matrix.from_raw(g)
    for kt in sorted({1, (k + 63) // 64}):
        for rule in (0, 1):
            d = grb.descriptor(direction=direction, rule=rule)
            lev = grb.msbfs(A, src, words_per_pass=min(kt, 8), desc=d).cpu().numpy().T
            st = grb.last_stats()
            assert np.array_equal(lev, ref), (kt, rule)
            assert st["iterations"] == ref.max() + 1
            pairs = np.bincount(ref[ref >= 0].ravel())[: len(st["frontier"])]
            assert st["frontier"] == pairs.tolist()
    for cap in (1, 5, 6, 7, 8, 9, 12, 20, 50):
        d = grb.descriptor(direction=direction, max_iter=cap)
        lev = grb.msbfs(A, src, desc=d).cpu().numpy().T
        assert np.array_equal(lev, np.where(ref <= cap, ref, -1)), cap


@pytest.mark.parametrize("step", [1, 3, 16])
def test_session_forms(grb, tails, step):
    g, adj, p, ends = tails
    k = 200
    ss = grb.MsbfsSession(grb.Matrix.from_raw(g), k)
    src = _sources(p, ends, 3 * k, 5)
    ref = oracle.msbfs(adj, src, nthreads=8)
    todo, free, busy, seen, turn = list(range(3 * k)), list(range(k)), {}, 0, 0
    while todo or busy:
        take = min(len(free), len(todo), (120, 1, 40)[turn % 3])  # joins in any state
        turn += 1
        if take:
            lanes, qs = free[:take], todo[:take]
            del free[:take], todo[:take]
            ss.join(lanes, src[qs])
            busy.update(zip(lanes, qs))
        done, _ = ss.step(step)
        if done:
            out = ss.extract(done).cpu().numpy()
            for lane, lev in zip(done, out):
                assert np.array_equal(lev, ref[busy[lane]]), (lane, turn)
                del busy[lane]
                seen += 1
            free += done
    assert seen == 3 * k
