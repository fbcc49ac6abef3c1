"""Bucketed SSSP in the multi-workgroup loops: one workgroup, several (ids that
follow the structure and shuffled ones, odd sizes), lists that overflow, the
queue loop above 64 workgroups, round caps and exchanges given up: distances
bit-equal to the oracle's, records within the cap."""
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


_CACHE = {}


def _graph(name):
    if name in _CACHE:
        return _CACHE[name]
    if name.startswith("grid"):
        r, c = {"grid_one": (180, 181), "grid_two": (181, 181), "grid_odd": (403, 257),
                "grid_shuffled": (300, 300), "grid_queue": (1447, 1447)}[name]
        g = graphgen.grid(r, c)
        if name == "grid_shuffled":
            p = np.random.default_rng(3).permutation(g.n).astype(np.int32)
            g = graphgen.from_edges(name, g.n, p[g.src], p[g.dst], g.w)
        src = [0, g.n // 2 + 7]
    else:  # 1 - 50 - 2500 vertices below one bucket, then a path: near lists overflow
        n = 100003
        up, mid = np.arange(10, 60), np.arange(40000, 42500)
        path = np.arange(n - 500, n)
        s = np.concatenate([np.zeros(50, int), up[np.arange(2500) % 50], [mid[-1]], path[:-1]])
        d = np.concatenate([up, mid, [path[0]], path[1:]])
        g = graphgen.from_edges(name, n, s, d, 1 + (s * 7 + d) % 64)
        src = [0]
    adj = oracle.Adjacency.from_raw(g)
    _CACHE[name] = (g, src, [oracle.sssp(adj, int(v))[0] for v in src])
    return _CACHE[name]


@pytest.mark.parametrize("flags", [0, 0x20], ids=["loop", "no_wait"])
@pytest.mark.parametrize("name", ["grid_one", "grid_two", "grid_odd", "grid_shuffled", "lists_full",
                                  "grid_queue"])
def test_delta_loop(grb, name, flags):
    g, sources, refs = _graph(name)
    A = grb.Matrix.from_raw(g)
    for s, ref in zip(sources, refs):
        for delta in ((7.5, 512.0, 1e6) if name != "grid_queue" else (512.0,)):
            dist = grb.sssp(A, int(s), delta=delta, desc=grb.descriptor(flags=flags))
            assert np.array_equal(dist.cpu().numpy(), ref), (name, s, delta)
        for cap in (1, 2, 40):
            d = grb.descriptor(flags=flags, max_iter=cap)
            got = grb.sssp(A, int(s), delta=64.0, desc=d).cpu().numpy()
            st = grb.last_stats()
            assert st["iterations"] <= cap
            assert np.all(got >= ref) and got[s] == 0
            if cap == 40:
                assert np.isfinite(got).sum() > 50


@pytest.mark.parametrize("count", [3000, 4096, 4200, 6000])
def test_delta_loop_long_lists(grb, count):
    """`count` vertices of one workgroup become pending together: near ones in
    a wide bucket, far ones in narrow buckets (lists of 4,096 and 3,072)."""
    n = 100003
    a, b = np.arange(10, 30), np.arange(1000, 2000)
    c = np.arange(40000, 40000 + count)
    path = np.arange(n - 300, n)
    s = np.concatenate([np.zeros(20, int), a[np.arange(1000) % 20], b[np.arange(count) % 1000],
                        [c[-1]], path[:-1]])
    d = np.concatenate([a, b, c, [path[0]], path[1:]])
    g = graphgen.from_edges(f"fan{count}", n, s, d, 1 + (s * 7 + d) % 64)
    ref = oracle.sssp(oracle.Adjacency.from_raw(g), 0)[0]
    A = grb.Matrix.from_raw(g)
    for delta in (7.5, 64.0, 1e6):
        dist = grb.sssp(A, 0, delta=delta)
        assert np.array_equal(dist.cpu().numpy(), ref), (count, delta)
