"""The workloads whose speed this framework is judged by, each one call (or one
driver run) through the public Python API on inputs made from a seed.

A case is a dict of plain values:
  kind   bfs | sssp | sssp_delta | pagerank | pagerank_adaptive | cc | msbfs |
         product (mxv / vxm) | tricount | mxm
  graph  rmat: R-MAT (0.57, 0.19, 0.19, 0.05) over n vertices, ef * n drawn
         edges, cleaned; symmetrised except for the PageRank kinds;
         grid: rows x cols 4-neighbour grid
  shuffled  R-MAT ids in random order (data as loaded) or as generated (low
         ids are the hubs)
and the options of the call.  Graphs are built on the GPU with torch; matrix
preparation and workspaces are made once, as a program that keeps its graph does.
"""
from __future__ import annotations

import math

import torch

import paper_1908_01407_amd as grb

DEV = "cuda"


# ---- the cases ------------------------------------------------------------------

def listed():
    return [
        # interactive query on a small graph: launches and read-backs are all of it
        dict(name="bfs_rmat14", kind="bfs", graph="rmat", n=1 << 14, ef=16, shuffled=False,
             rule="paper", parents=True),
        # the headline graph, from any source, levels and parents
        dict(name="bfs_rmat22", kind="bfs", graph="rmat", n=1 << 22, ef=16, shuffled=False,
             rule="exact", parents=True),
        # hop counts on a road-like network: thousands of small levels
        dict(name="bfs_grid3000", kind="bfs", graph="grid", rows=3000, cols=3000, rule="paper",
             parents=True),
        # weighted distances on a social-network-like graph
        dict(name="sssp_rmat22", kind="sssp", graph="rmat", n=1 << 22, ef=16, shuffled=False,
             rule="exact"),
        # weighted distances on a road-like network, ragged extents
        dict(name="sssp_delta_grid", kind="sssp_delta", graph="grid", rows=2003, cols=1009,
             delta=512.0),
        # ranking of a directed web-like graph in single precision
        dict(name="pagerank_f32_rmat22", kind="pagerank", graph="rmat", n=1 << 22, ef=16,
             shuffled=False, dtype="f32", tol=1e-6),
        # ranking in double precision with converged vertices frozen, ids as loaded
        dict(name="pr_adaptive_f64_rmat20", kind="pagerank_adaptive", graph="rmat", n=1 << 20,
             ef=16, shuffled=True, dtype="f64", tol=1e-6, eps=1e-4),
        # components of a large sparse graph
        dict(name="cc_rmat22", kind="cc", graph="rmat", n=1 << 22, ef=16, shuffled=False),
        # a batch of hop-count queries answered together
        dict(name="msbfs_rmat20_k64", kind="msbfs", graph="rmat", n=1 << 20, ef=16, shuffled=False,
             k=64, rule="paper"),
        # one masked frontier expansion, the step of user-written traversals
        dict(name="mxv_or_rmat22", kind="product", graph="rmat", n=1 << 22, ef=16, shuffled=False,
             call="mxv", semiring="lor_land", density=0.01, form="bitmap", mask="comp_struct",
             mask_density=0.5, replace=True, accum=""),
        # one dense weighted product (SpMV), the step of iterative solvers
        dict(name="mxv_plus_f32_rmat20", kind="product", graph="rmat", n=1000003, ef=16,
             shuffled=True, call="mxv", semiring="plus_times_fp32", density=1.0, form="bitmap",
             mask="", mask_density=0.0, replace=False, accum=""),
        # triangle count of a social-network-like graph
        dict(name="tricount_rmat20", kind="tricount", graph="rmat", n=1 << 20, ef=16,
             shuffled=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["bfs", "bfs", "bfs_grid", "sssp", "sssp_delta", "pagerank",
                       "pagerank_adaptive", "cc", "msbfs", "product", "product", "product",
                       "tricount", "mxm"])
    c = dict(kind=kind)
    if kind in ("bfs_grid", "sssp_delta"):
        c.update(kind="bfs" if kind == "bfs_grid" else kind, graph="grid", rows=_log(rng, 60, 2000),
                 cols=_log(rng, 60, 2000))
        if kind == "bfs_grid":
            c.update(rule=rng.choice(["paper", "exact"]), parents=rng.random() < 0.7)
        else:
            c.update(delta=float(rng.choice([128, 256, 512])))
        return c
    top = {"msbfs": 20, "tricount": 20, "mxm": 18, "pagerank_adaptive": 21}.get(kind, 22)
    c.update(graph="rmat", n=_log(rng, 1 << 14, 1 << top), ef=rng.randint(6, 16),
             shuffled=rng.random() < 0.5)
    if kind == "bfs":
        c.update(rule=rng.choice(["paper", "exact"]), parents=rng.random() < 0.7)
    elif kind == "sssp":
        c.update(rule=rng.choice(["paper", "exact"]))
    elif kind == "pagerank":
        c.update(dtype=rng.choice(["f32", "f64"]), tol=1e-6)
    elif kind == "pagerank_adaptive":
        c.update(dtype="f64", tol=1e-6, eps=rng.choice([1e-3, 1e-4, 1e-5]))
    elif kind == "msbfs":
        c.update(k=_log(rng, 2, max(2, min(512, (1 << 26) // c["n"]))),
                 rule=rng.choice(["paper", "exact"]))
    elif kind == "product":
        sr = rng.choice(["lor_land", "lor_land", "plus_times_fp32", "plus_times_fp64",
                         "min_plus_fp32", "min_second_int32"])
        dens = math.exp(rng.uniform(math.log(1e-4), 0.0))
        mask = rng.choice(["", "struct", "comp_struct", "value", "comp_value"])
        acc = {"lor_land": "lor", "min_plus_fp32": "min", "min_second_int32": "min"}.get(sr, "")
        c.update(call=rng.choice(["mxv", "vxm"]), semiring=sr, density=dens,
                 form=rng.choice(["bitmap", "bitmap", "list"]), mask=mask,
                 mask_density=rng.uniform(0.05, 0.9) if mask else 0.0,
                 replace=bool(mask) and rng.random() < 0.5, accum=acc if rng.random() < 0.4 else "")
    elif kind == "mxm":
        c.update(semiring=rng.choice(["plus_pair_int32", "plus_times_fp32"]))
    return c


# ---- graphs -----------------------------------------------------------------------

def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + salt) % (1 << 62))


def _rmat_edges(case, seed):
    n, m = case["n"], case["n"] * case["ef"]
    g = _gen(seed, 1)
    src = torch.zeros(m, dtype=torch.int32, device=DEV)
    dst = torch.zeros(m, dtype=torch.int32, device=DEV)
    for _ in range(max(1, (n - 1).bit_length())):
        x = torch.rand(m, generator=g, device=DEV)
        rb = x >= 0.76
        cb = ((x >= 0.57) & ~rb) | (x >= 0.95)
        src.mul_(2).add_(rb)
        dst.mul_(2).add_(cb)
    src, dst = src.remainder_(n), dst.remainder_(n)
    if case["shuffled"]:
        perm = torch.randperm(n, generator=_gen(seed, 2), device=DEV).to(torch.int32)
        src, dst = perm[src.long()], perm[dst.long()]
    return src, dst


def _keys(n, src, dst, symmetrise):
    """Sorted distinct row * n + column keys without self-loops."""
    src, dst = src.long(), dst.long()
    key = src * n + dst
    if symmetrise:
        key = torch.cat([key, dst * n + src])
        keep = torch.cat([src != dst, src != dst])
    else:
        keep = src != dst
    key = key[keep].sort().values
    if key.numel() > 1:
        key = key[torch.cat([torch.ones(1, dtype=torch.bool, device=DEV), key[1:] != key[:-1]])]
    return key


def _csr(n, key):
    row = key // n
    rp = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.bincount(row, minlength=n).cumsum(0).to(torch.int32)
    return rp, (key - row * n).to(torch.int32)


def _weights(n, key, seed):
    """Whole weights 1..64, the same for (u, v) and (v, u)."""
    r = key // n
    c = key - r * n
    h = torch.minimum(r, c) * 0x9E3779B1 + torch.maximum(r, c) * 0x85EBCA77 + int(seed) * 0xC2B2AE3D
    h = (h ^ (h >> 15)) * 0x2C1B3C6D
    return ((h >> 17) & 63).add_(1).to(torch.float32)


def _grid_keys(case):
    R, C = case["rows"], case["cols"]
    n = R * C
    v = torch.arange(n, device=DEV)
    right, down = v[v % C < C - 1], v[: (R - 1) * C]
    src = torch.cat([right, down])
    dst = torch.cat([right + 1, down + C])
    return _keys(n, src, dst, True)


def _graph(case, seed):
    """(n, keys of A) of the case's graph."""
    if case["graph"] == "grid":
        return case["rows"] * case["cols"], _grid_keys(case)
    src, dst = _rmat_edges(case, seed)
    return case["n"], _keys(case["n"], src, dst, not case["kind"].startswith("pagerank"))


def _lower_keys(n, key):
    """Strict lower triangle after renumbering by decreasing degree."""
    r, c = key // n, key - (key // n) * n
    order = torch.argsort(torch.bincount(r, minlength=n), descending=True, stable=True)
    rank = torch.empty_like(order)
    rank[order] = torch.arange(n, device=DEV)
    r, c = rank[r], rank[c]
    keep = c < r
    return (r[keep] * n + c[keep]).sort().values


def _sources(n, key, k, seed):
    """k sources among the vertices with edges."""
    live = torch.unique_consecutive(key // n)
    pick = torch.randint(live.numel(), (k,), generator=_gen(seed, 3), device=DEV)
    return live[pick].to(torch.int32)


def _bits(n, density, seed, salt):
    if density >= 1.0:
        return torch.ones(n, dtype=torch.bool, device=DEV)
    return torch.rand(n, generator=_gen(seed, salt), device=DEV) < density


def _words(bits):
    """Presence words (bit i % 64 of word i / 64) of a boolean vector."""
    n = bits.numel()
    pad = torch.zeros((n + 63) // 64 * 64, dtype=torch.int64, device=DEV)
    pad[:n] = bits
    return (pad.view(-1, 64) << torch.arange(64, device=DEV)).sum(1)


_DT = {"lor_land": torch.uint8, "min_second_int32": torch.int32, "plus_times_fp64": torch.float64}


def _operands(case, seed, n):
    """(u values, u presence, mask values, mask presence, old w values and presence)."""
    dt = _DT.get(case["semiring"], torch.float32)
    ub = _bits(n, case["density"], seed, 4)
    if case["semiring"] == "lor_land":
        u = torch.ones(n, dtype=dt, device=DEV)
        w = torch.ones(n, dtype=dt, device=DEV)
    elif case["semiring"] == "min_second_int32":
        u = torch.arange(n, dtype=dt, device=DEV)
        w = torch.arange(n, dtype=dt, device=DEV)
    else:
        u = torch.rand(n, generator=_gen(seed, 5), device=DEV, dtype=dt)
        w = torch.rand(n, generator=_gen(seed, 6), device=DEV, dtype=dt)
        if case["semiring"].startswith("min"):
            u, w = u * 64, w * 64 + 8
    mb = _bits(n, case["mask_density"], seed, 7) if case["mask"] else None
    mv = (torch.rand(n, generator=_gen(seed, 8), device=DEV) < 0.8).to(torch.uint8)
    wb = _bits(n, 0.3, seed, 9)
    return u, ub, mv, mb, torch.where(wb, w, torch.zeros_like(w)), wb


def _vector(n, values, bits, form="bitmap"):
    v = grb.Vector(n, values.dtype, device=DEV, sparse=form == "list")
    v.values[:n].copy_(values)
    v.bitmap.copy_(_words(bits))
    if form == "list":
        idx = bits.nonzero().flatten().to(torch.int32)
        v.indices[: idx.numel()].copy_(idx)
        v.count.fill_(idx.numel())
    return v


def _value_weights(key, seed, dtype):
    return torch.rand(key.numel(), generator=_gen(seed, 10), device=DEV, dtype=dtype)


# ---- preparation, one pass ----------------------------------------------------------

def prepare(case, seed):
    n, key = _graph(case, seed)
    kind = case["kind"]
    s = dict(case=case, n=n)
    rule = grb.SWITCH_EXACT if case.get("rule") == "exact" else grb.SWITCH_PAPER
    s["desc"] = grb.descriptor(rule=rule)
    if kind in ("tricount", "mxm"):
        low = _lower_keys(n, key)
        rp, ci = _csr(n, low)
        vals = _value_weights(low, seed, torch.float32) if case.get("semiring") == \
            "plus_times_fp32" else None
        s["A"] = grb.Matrix(n, n, rp, ci, vals, device=DEV)
        s["ws"] = grb.workspace(grb.OP_MXM, None, device=DEV)
        return s
    rp, ci = _csr(n, key)
    if kind.startswith("pagerank"):
        r = key // n
        trp, tci = _csr(n, ((key - r * n) * n + r).sort().values)
        s["A"] = grb.Matrix(n, n, rp, ci, None, trp, tci, device=DEV)
        s["dtype"] = torch.float64 if case["dtype"] == "f64" else torch.float32
        s["ws"] = grb.workspace(grb.OP_PAGERANK, s["A"], 2 if case["dtype"] == "f64" else 1)
        return s
    if kind == "product":
        vals = None
        if case["semiring"].startswith("plus_times"):
            vals = _sym_values(n, key, seed, _DT.get(case["semiring"], torch.float32))
        elif case["semiring"] == "min_plus_fp32":
            vals = _weights(n, key, seed)
        s["A"] = grb.Matrix(n, n, rp, ci, vals, symmetric=True, device=DEV)
        u, ub, mv, mb, w, wb = _operands(case, seed, n)
        s["u"] = _vector(n, u, ub, case["form"])
        s["mask"] = _vector(n, mv, mb) if mb is not None else None
        s["w"] = _vector(n, w, wb)
        flags = (grb.GRB_MASK_COMP if case["mask"].startswith("comp") else 0) | \
            (grb.GRB_MASK_STRUCT if case["mask"].endswith("struct") else 0) | \
            (grb.GRB_REPLACE if case["replace"] else 0)
        s["desc"] = grb.descriptor(flags=flags)
        s["ws"] = grb.workspace(grb.OP_MXV, s["A"])
        return s
    vals = _weights(n, key, seed) if kind.startswith("sssp") else None
    A = s["A"] = grb.Matrix(n, n, rp, ci, vals, symmetric=True, device=DEV)
    if kind == "bfs":
        s["source"] = int(_sources(n, key, 1, seed)[0])
        s["ws"] = grb.workspace(grb.OP_BFS, A)
        lev = torch.empty(n, dtype=torch.int32, device=DEV)
        s["out"] = (lev, torch.empty_like(lev) if case["parents"] else None)
    elif kind.startswith("sssp"):
        s["source"] = int(_sources(n, key, 1, seed)[0])
        s["ws"] = grb.workspace(grb.OP_SSSP, A)
    elif kind == "cc":
        s["ws"] = grb.workspace(grb.OP_CC, A)
    else:  # msbfs
        s["sources"] = _sources(n, key, case["k"], seed)
        s["ws"] = grb.workspace(grb.OP_MSBFS, A, case["k"])
        s["levels"] = torch.empty((n, case["k"]), dtype=torch.int32, device=DEV)
    return s


def _sym_values(n, key, seed, dtype):
    """Values in [0, 1), the same for (u, v) and (v, u)."""
    r = key // n
    c = key - r * n
    h = torch.minimum(r, c) * 0x9E3779B1 + torch.maximum(r, c) * 0x85EBCA77 + int(seed) * 0xC2B2AE3D
    h = (h ^ (h >> 15)) * 0x2C1B3C6D
    return ((h >> 9) & 0xFFFFFF).to(dtype) / (1 << 24)


def run(s):
    c, A = s["case"], s["A"]
    kind = c["kind"]
    if kind == "bfs":
        lev, par = grb.bfs(A, s["source"], parents=c["parents"], desc=s["desc"], ws=s["ws"],
                           out=s["out"])
        return (lev, par) if par is not None else (lev,)
    if kind == "sssp":
        return grb.sssp(A, s["source"], desc=s["desc"], ws=s["ws"])
    if kind == "sssp_delta":
        return grb.sssp(A, s["source"], delta=c["delta"], ws=s["ws"])
    if kind == "pagerank":  # the last change is at rounding level in fp32: not an output
        p, it, _ = grb.pagerank(A, dtype=s["dtype"], tol=c["tol"], ws=s["ws"])
        return p, it
    if kind == "pagerank_adaptive":
        p, it, _, active = grb.pagerank_adaptive(A, c["eps"], dtype=s["dtype"], tol=c["tol"],
                                                 ws=s["ws"])
        return p, it, active
    if kind == "cc":
        return grb.cc(A, ws=s["ws"])
    if kind == "msbfs":
        return grb.msbfs(A, s["sources"], desc=s["desc"], ws=s["ws"], levels=s["levels"])
    if kind == "tricount":
        return grb.tricount(A, ws=s["ws"])
    if kind == "mxm":
        return grb.mxm_masked(A, A, A, c["semiring"], ws=s["ws"])
    accum = c["accum"] or None
    if c["call"] == "mxv":
        grb.mxv(s["w"], s["mask"], accum, c["semiring"], A, s["u"], desc=s["desc"], ws=s["ws"])
    else:
        grb.vxm(s["w"], s["mask"], accum, c["semiring"], s["u"], A, desc=s["desc"], ws=s["ws"])
    return s["w"].values, s["w"].bitmap


# ---- what a pass cannot do without ----------------------------------------------------

def _sizes(case):
    """(vertices, stored entries): distinct entries of R-MAT are about 81 % of
    the drawn ones at 2^14 vertices and 96 % at 2^22."""
    if case["graph"] == "grid":
        R, C = case["rows"], case["cols"]
        return R * C, 2 * (R * (C - 1) + C * (R - 1))
    n = case["n"]
    m = n * case["ef"] * (1 if case["kind"].startswith("pagerank") else 2)
    return n, int(m * min(0.97, 0.81 + 0.018 * (math.log2(n) - 14)))


def work(case):
    n, nnz = _sizes(case)
    kind = case["kind"]
    if kind == "bfs":  # row starts, one found neighbour per vertex, the outputs
        return dict(bytes=4 * n + 4 * n + (8 if case["parents"] else 4) * n, flops=0)
    if kind.startswith("sssp"):  # every entry with its weight once, the distances
        return dict(bytes=4 * n + 8 * nnz + 4 * n, flops=2 * nnz)
    if kind.startswith("pagerank"):  # about ten sweeps of the column ids and vectors
        e = 8 if case["dtype"] == "f64" else 4
        it = 10
        return dict(bytes=it * (4 * nnz + 8 * n + 4 * e * n), flops=it * 2 * nnz)
    if kind == "cc":
        return dict(bytes=4 * n + 4 * nnz + 4 * n, flops=0)
    if kind == "msbfs":  # the entries once, the level block
        return dict(bytes=4 * n + 4 * nnz + 4 * n * case["k"], flops=0)
    if kind in ("tricount", "mxm"):  # the lower triangle once, the results
        out = 8 if kind == "tricount" else 4 * (nnz // 2)
        return dict(bytes=4 * n + 2 * nnz + out, flops=0)
    e = {torch.uint8: 1, torch.float64: 8}.get(_DT.get(case["semiring"], torch.float32), 4)
    ev = e if case["semiring"].startswith(("plus", "min_plus")) else 0
    touched = min(1.0, case["density"] * 1.0)
    return dict(bytes=int(touched * ((4 + ev) * nnz + (8 + e) * n) + 4 * n / 8 + e * n),
                flops=2 * int(touched * nnz))


# ---- references in 64 bits --------------------------------------------------------------

def _exact_grid_sssp(case, seed):
    R, C = case["rows"], case["cols"]
    n = R * C
    key = _grid_keys(case)
    src = int(_sources(n, key, 1, seed)[0])
    r = key // n
    d = key - r * n - r
    w = _weights(n, key, seed).double()
    right = torch.full((R, C), math.inf, dtype=torch.float64, device=DEV)
    down = torch.full((R, C), math.inf, dtype=torch.float64, device=DEV)
    right.view(-1)[r[d == 1]] = w[d == 1]
    down.view(-1)[r[d == C]] = w[d == C]
    dist = torch.full((R, C), math.inf, dtype=torch.float64, device=DEV)
    dist.view(-1)[src] = 0
    while True:
        old = dist.clone()
        for _ in range(128):
            t = dist.clone()
            t[:, 1:] = torch.minimum(t[:, 1:], dist[:, :-1] + right[:, :-1])
            t[:, :-1] = torch.minimum(t[:, :-1], dist[:, 1:] + right[:, :-1])
            t[1:] = torch.minimum(t[1:], dist[:-1] + down[:-1])
            t[:-1] = torch.minimum(t[:-1], dist[1:] + down[:-1])
            dist = t
        if torch.equal(old, dist):
            return dist.view(-1)


def _exact_sssp(case, seed):
    n, key = _graph(case, seed)
    src = int(_sources(n, key, 1, seed)[0])
    r = key // n
    c = key - r * n
    w = _weights(n, key, seed).double()
    dist = torch.full((n,), math.inf, dtype=torch.float64, device=DEV)
    dist[src] = 0
    while True:
        new = dist.scatter_reduce(0, c, dist[r] + w, "amin")
        if torch.equal(new, dist):
            return dist
        dist = new


def _exact_pagerank(case, seed):
    n, key = _graph(case, seed)
    r = key // n
    c = key - r * n
    od = torch.bincount(r, minlength=n).double()
    dang = od == 0
    inv = torch.where(dang, torch.zeros_like(od), 1.0 / od.clamp(min=1))
    p = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
    live = torch.ones(n, dtype=torch.bool, device=DEV)
    it, adaptive = 0, case["kind"] == "pagerank_adaptive"
    while it < 50:
        t = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, c, (p * inv)[r])
        q = 0.15 / n + 0.85 * (t + float(p[dang].sum()) / n)
        if adaptive:
            q = torch.where(live, q, p)
            live = live & ((q - p).abs() > case["eps"] * p)
        delta = float((q - p).abs().sum())
        p = q
        it += 1
        if delta < case["tol"] or (adaptive and not bool(live.any())):
            break
    return [p, None, None] if adaptive else [p, None]


def _exact_product(case, seed):
    n, key = _graph(case, seed)
    r = key // n
    c = key - r * n
    plus = case["semiring"].startswith("plus")
    dt = _DT.get(case["semiring"], torch.float32)
    a = (_sym_values(n, key, seed, dt) if plus else _weights(n, key, seed)).double()
    u, ub, mv, mb, w, wb = _operands(case, seed, n)
    keep = ub[c]
    r, c, a = r[keep], c[keep], a[keep]
    has = torch.zeros(n, dtype=torch.bool, device=DEV)
    has[r] = True
    if plus:
        t = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, r, a * u.double()[c])
    else:
        t = torch.full((n,), math.inf, dtype=torch.float64, device=DEV)
        t = t.scatter_reduce(0, r, a + u.double()[c], "amin")
    allowed = torch.ones_like(has)
    if mb is not None:
        m = mb & (mv != 0) if case["mask"].endswith("value") else mb
        allowed = ~m if case["mask"].startswith("comp") else m
    old = w.double()
    if case["accum"]:
        t = torch.where(has & wb, torch.minimum(old, t), torch.where(has, t, old))
        has = has | wb
    # entries that the product leaves absent keep their stored value
    return [torch.where(allowed & has, t, old), None]


def exact(case, seed):
    kind = case["kind"]
    if kind == "sssp_delta":
        return _exact_grid_sssp(case, seed)
    if kind == "sssp":
        return _exact_sssp(case, seed)
    if kind.startswith("pagerank"):
        return _exact_pagerank(case, seed)
    if kind == "product" and case["semiring"].startswith(("plus_times", "min_plus")):
        return _exact_product(case, seed)
    return None
