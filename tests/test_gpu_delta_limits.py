"""Bucketed SSSP where a bucket's limit, rounded, would not lie above the distance
it was taken from: the round kernel (rows longer than 64 entries, or a loop that
handed over), the owner loop and the queue loop all end, with exact distances.
Rounds are capped so that a search without end would stop and fail."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def grb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_01407_amd as g
    return g


@pytest.mark.parametrize("flags", [0, 0x20], ids=["loop", "no_wait"])
@pytest.mark.parametrize("delta,step", [(0.17527635, 1.2269344), (1e-5, 200.0), (1e-3, 3e9)])
@pytest.mark.parametrize("n,leaves", [(1000, 100), (1000, 10), (100003, 10), (2200003, 10)],
                         ids=["rounds", "one_group", "groups", "queue"])
def test_delta_limits(grb, n, leaves, delta, step, flags):
    # source 0: `leaves` neighbours near it, then a path whose first edge is `step`
    path = np.linspace(n // 2, n - 1, 6).astype(np.int64)
    s = np.concatenate([np.zeros(leaves + 1, np.int64), path[:-1]])
    d = np.concatenate([np.arange(1, leaves + 1), path])
    w = np.concatenate([np.full(leaves, 0.9 * delta), [step], np.full(5, step / 7)]).astype(np.float32)
    ref = np.full(n, np.inf, np.float32)
    ref[0] = 0
    for u, v, x in zip(s, d, w):
        ref[v] = ref[u] + x
    key = np.concatenate([s * n + d, d * n + s])
    o = np.argsort(key)
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(np.bincount(key // n, minlength=n))
    A = grb.Matrix(n, n, rp, (key[o] % n).astype(np.int32), np.concatenate([w, w])[o], symmetric=True)
    dist = grb.sssp(A, 0, delta=delta, desc=grb.descriptor(max_iter=500, flags=flags))
    assert np.array_equal(dist.cpu().numpy(), ref)
    assert grb.last_stats()["iterations"] < 100
