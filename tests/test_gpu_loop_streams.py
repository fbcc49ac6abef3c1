"""Multi-workgroup level loops beside other work on the device: BFS and bucketed
SSSP loops of several workgroups that overlap each other, and loops that start
while other streams keep every CU busy, which must wait for their workgroups to
become resident instead of continuing with a launch per level."""
import threading

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


@pytest.fixture(scope="module")
def grid(grb):
    g = graphgen.grid(701, 699)  # 8 workgroups for BFS, 15 for bucketed SSSP
    adj = oracle.Adjacency.from_raw(g)
    src = [0, 245000, 489998]
    return (grb.Matrix.from_raw(g), src, [oracle.bfs(adj, v) for v in src],
            [oracle.sssp(adj, v)[0] for v in src])


def _run(jobs):
    errors = []

    def guard(f, *a):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                f(*a)
        except Exception as e:
            errors.append(repr(e))

    threads = [threading.Thread(target=guard, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_loops_overlap(grb, grid):
    A, src, bfs_ref, sssp_ref = grid
    torch.cuda.synchronize()

    def work(seed):
        wsb, wss = grb.workspace(grb.OP_BFS, A), grb.workspace(grb.OP_SSSP, A)
        s = torch.cuda.current_stream()
        for i in range(4):
            k = (seed + i) % 3
            if (seed + i) % 2:
                lev, par = grb.bfs(A, src[k], ws=wsb, stream=s)
                s.synchronize()
                assert np.array_equal(lev.cpu().numpy(), bfs_ref[k][0]), ("levels", seed, i)
                assert np.array_equal(par.cpu().numpy(), bfs_ref[k][1]), ("parents", seed, i)
            else:
                dist = grb.sssp(A, src[k], delta=256.0, ws=wss, stream=s)
                s.synchronize()
                assert np.array_equal(dist.cpu().numpy(), sssp_ref[k]), ("sssp", seed, i)

    _run([(work, t) for t in range(4)])


def test_loops_beside_busy_streams(grb, grid):
    A, src, bfs_ref, sssp_ref = grid
    # 2^21 vertices, 64M entries: a PageRank iteration fills the chip
    n, m = 1 << 21, 1 << 26
    rp = (torch.arange(n + 1, device="cuda") * (m // n)).to(torch.int32)
    ci = torch.randint(n, (m,), device="cuda", dtype=torch.int32, generator=torch.Generator(
        device="cuda").manual_seed(3)).view(n, -1).sort(1).values.flatten()
    B = grb.Matrix(n, n, rp, ci, None, symmetric=True)
    torch.cuda.synchronize()
    stop, up = threading.Event(), threading.Barrier(3)

    def busy():
        ws, s = grb.workspace(grb.OP_PAGERANK, B, 1), torch.cuda.current_stream()
        up.wait()
        while not stop.is_set():
            grb.pagerank(B, tol=0.0, max_iter=16, ws=ws, stream=s)

    def loops():
        try:
            wsb, wss = grb.workspace(grb.OP_BFS, A), grb.workspace(grb.OP_SSSP, A)
            s = torch.cuda.current_stream()
            up.wait()
            for i in range(6):
                k = i % 3
                lev, _ = grb.bfs(A, src[k], ws=wsb, stream=s)
                assert grb.last_stats()["launches"] == 1, ("bfs handed over", i)
                assert np.array_equal(lev.cpu().numpy(), bfs_ref[k][0]), ("levels", i)
                dist = grb.sssp(A, src[k], delta=256.0, ws=wss, stream=s)
                assert grb.last_stats()["launches"] == 1, ("sssp handed over", i)
                assert np.array_equal(dist.cpu().numpy(), sssp_ref[k]), ("sssp", i)
        finally:
            stop.set()

    _run([(busy,), (busy,), (loops,)])
