"""Round caps of bucketed SSSP where a round sends more messages to one workgroup
than a box holds, or leaves more near vertices than a list holds: every relaxation
of the rounds before the cap counts."""
import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def grb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_01407_amd as g
    return g


@pytest.mark.parametrize("flags", [0, 0x20], ids=["loop", "no_wait"])
@pytest.mark.parametrize("count", [4000, 4600, 6000, 9000])
def test_capped_round_with_full_boxes(grb, count, flags):
    """Layers of 1, 20, 1000 and `count` vertices, then a path: in one bucket
    round k relaxes the edges that leave layer k, so a run of `cap` rounds
    knows the exact distances of layers 0 to cap (workgroups that gave an
    exchange up may know some beyond).  A box of 4 workgroups and 100,003
    vertices holds 4,687 messages, a list 4,096 vertices."""
    n = 100003
    a, b = np.arange(10, 30), np.arange(1000, 2000)
    c = np.arange(40000, 40000 + count)
    path = np.arange(n - 300, n)
    s = np.concatenate([np.zeros(20, int), a[np.arange(1000) % 20], b[np.arange(count) % 1000],
                        [c[-1]], path[:-1]])
    d = np.concatenate([a, b, c, [path[0]], path[1:]])
    w = 1 + (s * 7 + d) % 64
    A = grb.Matrix.from_raw(graphgen.from_edges(f"capfan{count}", n, s, d, w))
    ref = np.full(n, np.inf, np.float32)  # the graph is a tree: one path to every vertex
    layer = np.full(n, np.iinfo(np.int32).max)
    ref[0] = layer[0] = 0
    for u, v, x in zip(s, d, w):  # listed in the order of the layers
        ref[v], layer[v] = ref[u] + x, layer[u] + 1
    for cap in (1, 2, 3, 4, 5, 40):
        got = grb.sssp(A, 0, delta=1e6, desc=grb.descriptor(max_iter=cap, flags=flags))
        got = got.cpu().numpy()
        assert np.array_equal(got[layer <= cap], ref[layer <= cap]), cap
        assert np.all((got == ref) | np.isinf(got)), cap
