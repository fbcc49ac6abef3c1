"""The level loops of BFS and bucketed SSSP with the workgroup counts of large
graphs, on small ones: up to 256 workgroups (several exchange records a lane) and
visited bits in device memory for BFS, up to 64 workgroups for bucketed SSSP; ids
that follow the structure and shuffled ones, odd sizes, workgroups that own
nothing, full boxes and queues, level caps and exchanges given up: against the
oracle."""
import ctypes

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


def _ws(grb, op, A, groups):
    b = ctypes.c_size_t()
    grb.check(grb.grb_loop_workspace_size(op, A.handle, groups, ctypes.byref(b)))
    return torch.empty(b.value, dtype=torch.uint8, device="cuda").fill_(0xA5)


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


def _bfs(grb, A, s, groups, dev, desc, ws):
    lev = torch.empty(A.nrows, dtype=torch.int32, device="cuda")
    par = torch.empty_like(lev)
    grb.check(grb.grb_bfs_loop(_p(lev), _p(par), A.handle, int(s), groups, dev, ctypes.byref(desc),
                               _p(ws), ws.numel(), None), "grb_bfs_loop")
    return lev.cpu().numpy(), par.cpu().numpy()


_CACHE = {}


def _graph(name):
    if name in _CACHE:
        return _CACHE[name]
    if name.startswith("grid"):
        r, c = {"grid": (231, 233), "grid_wide": (40, 1501), "grid_shuffled": (200, 200),
                "grid_tiny": (9, 11)}[name]
        g = graphgen.grid(r, c)
        if name == "grid_shuffled":
            p = np.random.default_rng(3).permutation(g.n).astype(np.int32)
            g = graphgen.from_edges(name, g.n, p[g.src], p[g.dst], g.w)
        src = [0, g.n // 2 + 7]
    else:  # layers of 1, 50, 3000 and 6000 vertices, then a path; ids in order or shuffled
        n = 60001
        lay = [np.arange(1), np.arange(10, 60), np.arange(20000, 23000), np.arange(40000, 46000)]
        path = np.concatenate([lay[-1][-1:], np.arange(n - 300, n)])
        s = np.concatenate([u[np.arange(v.size) % u.size] for u, v in zip(lay, lay[1:])] + [path[:-1]])
        d = np.concatenate(lay[1:] + [path[1:]])
        w = 1 + (s * 7 + d) % 64
        if name == "fan_shuffled":
            p = np.random.default_rng(5).permutation(n)
            s, d = p[s], p[d]
        g = graphgen.from_edges(name, n, s, d, w)
        src = [int(s[0])]
    adj = oracle.Adjacency.from_raw(g)
    _CACHE[name] = (g, src, [oracle.bfs(adj, v) for v in src], [oracle.sssp(adj, v)[0] for v in src])
    return _CACHE[name]


NAMES = ["grid", "grid_wide", "grid_shuffled", "grid_tiny", "fan", "fan_shuffled"]


@pytest.mark.parametrize("flags", [0, 0x20], ids=["loop", "no_wait"])
@pytest.mark.parametrize("groups,dev", [(16, 0), (64, 0), (65, 0), (128, 0), (256, 0), (1, 1), (5, 1),
                                        (64, 1)])
@pytest.mark.parametrize("name", NAMES)
def test_bfs_groups(grb, name, groups, dev, flags):
    g, sources, refs, _ = _graph(name)
    A = grb.Matrix.from_raw(g, weights=False)
    ws = _ws(grb, grb.OP_BFS, A, groups)
    for s, (ref_lev, ref_par, nl) in zip(sources, refs):
        for rule in (0, 1):
            lev, par = _bfs(grb, A, s, groups, dev, grb.descriptor(rule=rule, flags=flags), ws)
            st = grb.last_stats()
            assert np.array_equal(lev, ref_lev) and np.array_equal(par, ref_par), (s, rule)
            assert st["iterations"] == nl
            assert st["frontier"] == np.bincount(ref_lev[ref_lev >= 0])[: len(st["frontier"])].tolist()
        for cap in (1, 2, 3, 4, 7, 100):
            lev, _ = _bfs(grb, A, s, groups, dev, grb.descriptor(max_iter=cap, flags=flags), ws)
            assert np.array_equal(lev, np.where(ref_lev <= cap, ref_lev, -1)), (s, cap)


@pytest.mark.parametrize("flags", [0, 0x20], ids=["loop", "no_wait"])
@pytest.mark.parametrize("groups", [8, 33, 64])
@pytest.mark.parametrize("name", [n for n in NAMES if n != "grid_tiny"])
def test_delta_groups(grb, name, groups, flags):
    g, sources, _, refs = _graph(name)
    A = grb.Matrix.from_raw(g)
    ws = _ws(grb, grb.OP_SSSP, A, groups)
    for s, ref in zip(sources, refs):
        for delta in (7.5, 64.0, 512.0, 1e6):
            dist = torch.empty(A.nrows, dtype=torch.float32, device="cuda")
            d = grb.descriptor(flags=flags)
            grb.check(grb.grb_sssp_delta_loop(_p(dist), A.handle, int(s), delta, groups, ctypes.byref(d),
                                              _p(ws), ws.numel(), None), "grb_sssp_delta_loop")
            assert np.array_equal(dist.cpu().numpy(), ref), (s, delta)


def test_refused_shapes(grb):
    A = grb.Matrix.from_raw(_graph("grid_tiny")[0])
    ws = _ws(grb, grb.OP_SSSP, A, 64)
    x = torch.empty(A.nrows, dtype=torch.int32, device="cuda")
    for groups, dev in ((0, 0), (257, 0), (65, 1)):
        assert grb.grb_bfs_loop(_p(x), None, A.handle, 0, groups, dev, None, _p(ws), ws.numel(), None) == 4
    for groups in (0, 65, 64):  # 64: 99 vertices leave no room for a message a pair
        assert grb.grb_sssp_delta_loop(_p(x), A.handle, 0, 8.0, groups, None, _p(ws), ws.numel(), None) == 4
    assert grb.grb_bfs_loop(_p(x), None, A.handle, 0, 256, 0, None, _p(ws), 4096, None) == 9
