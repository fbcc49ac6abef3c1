"""Products over inputs that hold every index, all but one, or every index and
set bits beyond the last one; rows of one piece and of several; an OR push of
more tiles than it has copies of its temporary, with true, false and mixed
products on the same outputs."""
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


def _matrix(grb, n, lens, rng, vals):
    cols = [np.sort(rng.choice(n, size=k, replace=False)) for k in lens]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate(cols).astype(np.int32)
    v = vals(ci.size)
    row = np.repeat(np.arange(n), lens)
    o = np.lexsort((row, ci))
    trp = np.concatenate([[0], np.cumsum(np.bincount(ci, minlength=n))]).astype(np.int32)
    return grb.Matrix(n, n, rp, ci, v, trp, row[o].astype(np.int32), v[o]), row, ci, v


def _vector(grb, n, dt, values, present, junk=False):
    u = grb.Vector(n, dt)
    u.set({int(i): values[i].item() for i in np.flatnonzero(present)})
    if junk and n % 64:  # the padding of the last word
        u.bitmap[-1] |= -1 << (n % 64)
    return u


@pytest.mark.parametrize("n", [640, 701])
@pytest.mark.parametrize("semiring,dt", [("plus_times_fp32", "float32"), ("plus_times_fp64", "float64"),
                                         ("min_plus_fp32", "float32"), ("min_second_int32", "int32")])
@pytest.mark.parametrize("case", ["full", "junk", "one_missing"])
def test_dense_input(grb, n, semiring, dt, case):
    rng = np.random.default_rng(n)
    lens = [int(x) for x in rng.integers(0, 9, n)]
    for i, k in enumerate((0, 1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 600)):
        lens[7 * i] = k
    vdt = np.dtype(dt)
    # whole numbers: every order of the sums gives the same bits
    A, row, ci, v = _matrix(grb, n, lens, rng, lambda m: rng.integers(1, 9, m).astype(vdt))
    x = rng.integers(1, 9, n).astype(vdt)
    present = np.ones(n, bool)
    if case == "one_missing":
        present[n - 1 if n % 2 else 64] = False
    u = _vector(grb, n, getattr(torch, dt), x, present, case == "junk")
    keep = present[ci]
    has = np.zeros(n, bool)
    has[row[keep]] = True
    for direction in (0, 2):
        w = grb.Vector(n, getattr(torch, dt))
        grb.mxv(w, None, None, semiring, A, u, desc=grb.descriptor(direction=direction))
        if semiring.startswith("plus"):
            ref = np.zeros(n, vdt)
            np.add.at(ref, row[keep], v[keep] * x[ci[keep]])
        else:
            ref = np.full(n, np.iinfo(np.int32).max if dt == "int32" else np.inf, vdt)
            np.minimum.at(ref, row[keep], x[ci[keep]] + (v[keep] if semiring[4] == "p" else 0))
        assert w.to_dict() == {int(i): ref[i].item() for i in np.flatnonzero(has)}, direction


@pytest.mark.parametrize("masked", [False, True])
def test_or_push_copies(grb, masked):
    rng = np.random.default_rng(3)
    n = 6000
    lens = np.full(n, 40)
    lens[:4] = 3000  # 250,000 entries: about 250 tiles over eight copies
    A, row, ci, v = _matrix(grb, n, lens.tolist(), rng, lambda m: rng.integers(0, 2, m).astype(np.int32))
    x = rng.integers(0, 2, n).astype(np.uint8)
    present = rng.random(n) < 0.9
    u = _vector(grb, n, torch.uint8, x, present)
    # t(i) over the entries (j, i) of the pushed rows j: w = A^T u
    keep = present[row]
    has = np.zeros(n, bool)
    has[ci[keep]] = True
    tru = np.zeros(n, bool)
    tru[ci[keep & (v != 0) & (x[row] != 0)]] = True
    m = None
    if masked:
        allowed = rng.random(n) < 0.5
        m = _vector(grb, n, torch.int32, np.ones(n, np.int32), allowed)
        has &= allowed
    w = grb.Vector(n, torch.uint8)
    grb.vxm(w, m, None, "lor_land", u, A, desc=grb.descriptor(direction=1))
    got = w.to_dict()
    assert {i: bool(b) for i, b in got.items()} == {int(i): bool(tru[i]) for i in np.flatnonzero(has)}


@pytest.mark.parametrize("semiring,dt", [("min_plus_fp32", "float32"), ("min_plus_fp64", "float64"),
                                         ("min_second_int32", "int32")])
@pytest.mark.parametrize("hub", [1, 300])
def test_min_push(grb, semiring, dt, hub):
    """Pushes onto `hub` targets hit by every row and others hit by few, with
    products of either sign and some that equal the identity: a target whose
    only product is the identity is present all the same."""
    rng = np.random.default_rng(hub)
    n, vdt = 5000, np.dtype(dt)
    top = np.iinfo(np.int32).max if dt == "int32" else np.inf
    cols = [np.unique(np.concatenate([np.arange(hub), rng.integers(0, n, 12)])) for _ in range(n)]
    lens = [c.size for c in cols]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate(cols).astype(np.int32)
    row = np.repeat(np.arange(n), lens)
    v = rng.integers(-50, 50, ci.size).astype(vdt)
    x = rng.integers(-1000, 1000, n).astype(vdt)
    x[rng.random(n) < 0.3] = top
    x[rng.random(n) < 0.001] = top
    present = rng.random(n) < 0.4
    A = grb.Matrix(n, n, rp, ci, v)
    u = _vector(grb, n, getattr(torch, dt), x, present)
    w = grb.Vector(n, getattr(torch, dt))
    # w(j) = min over i of u(i) (x) A(i, j): the rows of A are pushed
    grb.mxv(w, None, None, semiring, A, u,
            desc=grb.descriptor(direction=1, flags=grb.GRB_TRAN_A))
    keep = present[row]
    ref = np.full(n, top, vdt)
    np.minimum.at(ref, ci[keep], x[row[keep]] + (v[keep] if semiring[4] == "p" else 0))
    has = np.zeros(n, bool)
    has[ci[keep]] = True
    assert (ref[has] == top).any()
    assert w.to_dict() == {int(i): ref[i].item() for i in np.flatnonzero(has)}
