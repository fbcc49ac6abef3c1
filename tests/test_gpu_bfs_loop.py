"""BFS level loop over several workgroups (low-degree graphs above 2^18
vertices): ids that follow the structure and shuffled ones, a box and a queue
that overflow, odd sizes, level caps, and exchanges given up: levels, parents,
iterations and the frontier record against the oracle."""
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


def _layers(n, sizes, start):
    """Layer i + 1 is spread over layer i (at most 60 children each); layer i
    holds consecutive ids from start[i]; a path of 300 follows the last one."""
    src, dst = [], []
    layers = [np.arange(b, b + k) for k, b in zip(sizes, start)]
    for up, down in zip(layers, layers[1:]):
        src.append(up[np.arange(down.size) % up.size])
        dst.append(down)
    path = np.concatenate([layers[-1][-1:], np.arange(n - 300, n)])
    src.append(path[:-1])
    dst.append(path[1:])
    return np.concatenate(src), np.concatenate(dst)


_CACHE = {}


def _graph(name):
    if name in _CACHE:
        return _CACHE[name]
    if name.startswith("grid"):
        r, c = (521, 523) if name == "grid_odd" else (520, 520)
        g = graphgen.grid(r, c, weights=False)
        if name == "grid_shuffled":
            p = np.random.default_rng(3).permutation(g.n).astype(np.int32)
            g = graphgen.from_edges(name, g.n, p[g.src], p[g.dst])
        src = [0, 260 * c + 100, g.n - 1]
    else:
        n = 300001
        if name == "box_full":  # 3000 targets of one workgroup found by another
            s, d = _layers(n, [1, 50, 3000], [0, 10, 200000])
        else:  # queue_full: 6000 targets of one workgroup, more than its queue
            s, d = _layers(n, [1, 20, 150, 6000], [0, 10, 1000, 200000 if name[-1] == "2" else 5000])
        g = graphgen.from_edges(name, n, s, d)
        src = [0]
    adj = oracle.Adjacency.from_raw(g)
    _CACHE[name] = (g, adj, src, [oracle.bfs(adj, int(v)) for v in src])
    return _CACHE[name]


@pytest.mark.parametrize("flags", [0, 0x20], ids=["loop", "no_wait"])
@pytest.mark.parametrize("name", ["grid_odd", "grid_even", "grid_shuffled", "box_full", "queue_full",
                                  "queue_full2"])
def test_bfs_loop(grb, name, flags):
    g, adj, sources, refs = _graph(name)
    A = grb.Matrix.from_raw(g, weights=False)
    off, _, _ = adj.arrays(weights=False)
    deg = np.diff(off)
    for s, (ref_lev, ref_par, nl) in zip(sources, refs):
        for rule in (0, 1):
            lev, par = grb.bfs(A, int(s), desc=grb.descriptor(rule=rule, flags=flags))
            st = grb.last_stats()
            assert np.array_equal(lev.cpu().numpy(), ref_lev), (name, s)
            assert np.array_equal(par.cpu().numpy(), ref_par), (name, s)
            assert st["iterations"] == nl
            k = len(st["frontier"])
            assert st["frontier"] == np.bincount(ref_lev[ref_lev >= 0])[:k].tolist()
            w = np.bincount(ref_lev[ref_lev >= 0], deg[ref_lev >= 0])[:k]
            assert st["edges"] == w.astype(int).tolist()
        for cap in (1, 2, 3, 7, 255, 256, 257):
            lev, _ = grb.bfs(A, int(s), parents=False, desc=grb.descriptor(max_iter=cap, flags=flags))
            want = np.where(ref_lev <= cap, ref_lev, -1)
            assert np.array_equal(lev.cpu().numpy(), want), (name, s, cap)
