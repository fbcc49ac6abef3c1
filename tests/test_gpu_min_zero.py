"""Min-plus products of -0.0 beside negative, zero and positive ones on the same
output: push and pull give the smallest value, whatever the order."""
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


@pytest.mark.parametrize("direction", [1, 2], ids=["push", "pull"])
@pytest.mark.parametrize("dt", ["float32", "float64"])
def test_negative_zero_products(grb, dt, direction):
    # row i of the matrix holds the weights of products[i], columns spread so
    # that a row's products come from several waves of a push; u = -0.0 keeps
    # a weight's own sign of zero
    n, rng = 4099, np.random.default_rng(1)
    pool = [-0.0, 0.0, -1.0, 1.0, -1e-42, 3.5, -7.25, np.inf]
    rows = [[x] for x in pool] + [[x, y] for x in pool for y in pool]
    rows += [list(rng.choice(pool, 40)) for _ in range(40)] + [[-0.0] * 300 + [-1.0]]
    rows += [[-2.0] + [-0.0] * 300]
    lens = np.zeros(n, int)
    lens[: len(rows)] = [len(r) for r in rows]
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lens[: len(rows)]])
    v = np.concatenate(rows).astype(dt)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    row = np.repeat(np.arange(n), lens)
    o = np.lexsort((row, ci))
    trp = np.concatenate([[0], np.cumsum(np.bincount(ci, minlength=n))]).astype(np.int32)
    A = grb.Matrix(n, n, rp, ci.astype(np.int32), v, trp, row[o].astype(np.int32), v[o])
    u = grb.Vector(n, getattr(torch, dt))
    u.fill(-0.0)
    sr = "min_plus_fp32" if dt == "float32" else "min_plus_fp64"
    for _ in range(4):
        w = grb.Vector(n, getattr(torch, dt))
        grb.mxv(w, None, None, sr, A, u, desc=grb.descriptor(direction=direction))
        got = w.to_dict()
        assert sorted(got) == list(range(len(rows)))
        for i, r in enumerate(rows):
            assert got[i] == min(np.asarray(r, dt).tolist()), (i, r)
