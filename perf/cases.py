"""The work that programs have this library do, as timed cases.

Every case is one call (or one batch of requests) through the public entry
points of ``paper_2107_12371_amd`` on a synthetic mesh matrix of a stated kind
and size.  ``listed()`` names the cases, ``draw(rng)`` gives one more of the
same ranges, ``prepare`` makes what a program holds before the call (resident
matrix, vectors, server), ``run`` is the call, ``work`` the bytes and
operations it cannot do without and ``exact`` its result in binary64 with
compensated sums, from plain torch.

The meshes are generated on the GPU from the seed:

* ``tet``    every cell of an nx x ny x nz box lattice cut into 6 tetrahedra
             (Kuhn's split); a row couples a tetrahedron to its face
             neighbours, at most five entries, as in the paper's matrices
             (49,336 to 775,058 rows, Table 1).
* ``knn``    jittered lattice, 4 to 6 nearest neighbours per cell, union
             (6.9 entries per row).
* ``hex27``  lattice cells with their face neighbours and each edge or vertex
             neighbour kept with probability 1/2 (7 to 27 entries per row).
* ``block``  3x3 blocks on a lattice: diagonal, faces and 0 to 4 directed
             extra neighbours within distance 2.

Scalar matrices are symmetric, off-diagonals -w with one w ~ U[0.5, 1.5) per
edge, diagonal sum(w) + 1e-3, as finite-volume Laplacians are; order ``rcm`` is
reverse Cuthill-McKee (the order a solver would use), ``random`` the worst one,
``natural`` the lattice's own.  ``long`` > 0 replaces that many rows by dense
coupling rows over 1/8 of the cells (a global constraint).
"""
import itertools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2107_12371_amd as spmv

DEV = "cuda"
VALUE_BYTES = {"f64": 8, "f32": 4, "f32v": 4, "bf16": 2}
VECTOR = {"f64": torch.float64, "f32v": torch.float64, "f32": torch.float32, "bf16": torch.float32}
CG_MODES = {"fp64": spmv.CG_FP64, "mixed": spmv.CG_MIXED_FP32, "jacobi": spmv.CG_PCG_JACOBI,
            "pcg_bf16": spmv.CG_PCG_BF16, "one_reduction": spmv.CG_FP64_ONE_REDUCTION}


def _product(name, mesh, dims, order, dtype="f64", k=1, long=0):
    return {"name": name, "op": "product", "mesh": mesh, "nx": dims[0], "ny": dims[1], "nz": dims[2],
            "order": order, "dtype": dtype, "k": k, "long": long}


def _solve(name, mesh, dims, mode, tol):
    return {"name": name, "op": "solve", "mesh": mesh, "nx": dims[0], "ny": dims[1], "nz": dims[2],
            "order": "rcm", "mode": mode, "tol": tol}


def listed():
    return [
        # one product inside a small solver (the paper's smallest mesh, 49K
        # cells): bound by the call and its launch
        _product("spmv_f64_tet_49k", "tet", (21, 14, 28), "rcm"),
        # an ordinary mesh, 2M cells; three of them do not fit the caches
        _product("spmv_f64_knn_2m", "knn", (126, 126, 126), "rcm"),
        # the same mesh as a generator numbered it: gathers all over x
        _product("spmv_f64_knn_2m_random", "knn", (126, 126, 126), "random"),
        # the large mesh of the library's benchmark, 16M cells
        _product("spmv_f64_hex27_16m", "hex27", (252, 252, 252), "rcm"),
        # reduced-precision products of mixed solvers, on odd sizes
        _product("spmv_f32_hex27_4m", "hex27", (161, 159, 157), "rcm", "f32"),
        _product("spmv_bf16_hex27_4m", "hex27", (159, 163, 155), "rcm", "bf16"),
        # eight right-hand sides at once (batched requests)
        _product("spmm_k8_hex27_4m", "hex27", (157, 161, 159), "rcm", "f64", 8),
        # momentum equations, three unknowns per cell
        _product("bsr3_f64_k1_4m", "block", (200, 200, 100), "natural"),
        _product("bsr3_f32_k4_1m7", "block", (121, 119, 117), "natural", "f32", 4),
        # a small solve, bound by its chain of launches
        _solve("cg_fp64_tet_49k", "tet", (21, 14, 28), "fp64", 1e-10),
        # a large solve in mixed precision, bound by memory
        _solve("cg_mixed_hex27_4m", "hex27", (160, 160, 160), "mixed", 1e-10),
        # a burst of product requests on resident matrices, host to host
        {"name": "serve_products", "op": "serve", "mesh": "hex27", "largest": 60, "matrices": 8, "requests": 16,
         "most_k": 16},
    ]


def _dims(rng, lo, hi):
    """Lattice edges for a log-uniform number of cells in [lo, hi]."""
    c = math.exp(rng.uniform(math.log(lo), math.log(hi))) ** (1.0 / 3.0)
    d = [max(3, int(round(c * rng.uniform(0.85, 1.15)))) for _ in range(3)]
    while d[0] * d[1] * d[2] > hi:
        d[d.index(max(d))] -= 1
    return tuple(d)


def draw(rng):
    what = rng.choice(["tet", "knn", "hex27", "hex27", "coupled", "spmm", "block", "block", "solve", "solve", "serve"])
    if what == "tet":
        c = _product("", "tet", _dims(rng, 1000, 200000), "rcm", rng.choice(["f64", "f64", "f32", "bf16"]))
    elif what == "knn":
        c = _product("", "knn", _dims(rng, 8000, 4e6), rng.choice(["rcm", "random", "natural"]),
                     rng.choice(["f64", "f64", "f32", "f32v"]))
    elif what == "hex27":
        c = _product("", "hex27", _dims(rng, 8000, 8e6), rng.choice(["rcm", "rcm", "natural"]),
                     rng.choice(["f64", "f64", "f32", "f32v", "bf16"]))
    elif what == "coupled":
        c = _product("", "knn", _dims(rng, 30000, 2e6), "rcm", "f64", 1, rng.randint(1, 16))
    elif what == "spmm":
        c = _product("", rng.choice(["hex27", "knn"]), _dims(rng, 8000, 2e6), "rcm", "f64",
                     rng.choice([2, 3, 4, 5, 8, 8, 12, 16]))
    elif what == "block":
        c = _product("", "block", _dims(rng, 3000, 2e6), "natural", rng.choice(["f64", "f32"]),
                     rng.choice([1, 1, 2, 3, 4, 8]))
    elif what == "solve":
        mode = rng.choice(list(CG_MODES))
        mesh = rng.choice(["tet", "hex27"])
        hi = {"tet": 130000, "hex27": 2e6}[mesh] if mode != "one_reduction" else {"tet": 33000, "hex27": 60000}[mesh]
        c = _solve("", mesh, _dims(rng, 500, hi), mode, rng.choice([1e-8, 1e-10]))
    else:
        c = {"name": "", "op": "serve", "mesh": "hex27", "largest": rng.randint(20, 60), "matrices": rng.randint(2, 8),
             "requests": rng.randint(4, 24), "most_k": rng.randint(1, 16)}
    del c["name"]
    return c


# ------------------------------------------------------------------ meshes

def _mix(a):
    """A 64-bit mixing function on int64 tensors (two multiply-xorshift
    rounds; the arithmetic wraps)."""
    a = (a ^ ((a >> 31) & 0x1FFFFFFFF)) * 0x4CF5AD432745937F
    a = (a ^ ((a >> 29) & 0x7FFFFFFFF)) * 0x2127599BF4325C37
    return a ^ ((a >> 32) & 0xFFFFFFFF)


def _unit(a):
    """U[0, 1) from mixed int64."""
    return ((a >> 11) & ((1 << 53) - 1)).to(torch.float64) * 2.0 ** -53


def _pair(i, j, seed, stream):
    """One mixed number per undirected pair."""
    lo, hi = torch.minimum(i, j), torch.maximum(i, j)
    return _mix(_mix(lo * 0x100000001B3 + hi) + (seed * 1000003 + stream) * 0x632BE59BD9B4E019 % (1 << 62))


_OFFSETS = [o for o in itertools.product((-1, 0, 1), repeat=3) if o != (0, 0, 0)]


def _lattice(nx, ny, nz, offsets):
    """Neighbour ids (n, len(offsets)) of a lattice, -1 outside it."""
    i = torch.arange(nx * ny * nz, device=DEV)
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    cols = []
    for dx, dy, dz in offsets:
        ok = (x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0) & (z + dz < nz)
        cols.append(torch.where(ok, i + dx + nx * (dy + ny * dz), -1))
    return torch.stack(cols, 1)


def _hex27(nx, ny, nz, seed):
    nb = _lattice(nx, ny, nz, _OFFSETS)
    i = torch.arange(nb.shape[0], device=DEV)
    for s, o in enumerate(_OFFSETS):
        if sum(abs(v) for v in o) > 1:
            drop = (_pair(i, nb[:, s].clamp(min=0), seed, 1) & (1 << 40)) != 0
            nb[:, s].masked_fill_(drop, -1)
    return nb


def _knn(nx, ny, nz, seed):
    nb = _lattice(nx, ny, nz, _OFFSETS)
    n = nb.shape[0]
    i = torch.arange(n, device=DEV)
    grid = torch.stack([i % nx, (i // nx) % ny, i // (nx * ny)], 1).to(torch.float64)
    jit = torch.stack([_unit(_mix(_mix(3 * i + c) + seed * 7919 + 11)) for c in range(3)], 1)
    pts = (grid + 0.7 * jit - 0.35).to(torch.float32)
    dist = torch.stack([torch.where(nb[:, s] >= 0, ((pts[nb[:, s].clamp(min=0)] - pts) ** 2).sum(1), torch.inf)
                        for s in range(len(_OFFSETS))], 1)
    near = torch.argsort(dist, 1)[:, :6]
    want = 4 + (_mix(i + seed * 31 + 5) >> 20) % 3
    mark = torch.zeros(nb.shape, dtype=torch.bool, device=DEV)
    mark.scatter_(1, near, torch.arange(6, device=DEV)[None, :] < want[:, None])
    mark &= nb >= 0
    both = mark.clone()
    for s in range(len(_OFFSETS)):  # the pair is kept if either end chose it
        both[:, s] |= mark[nb[:, s].clamp(min=0), len(_OFFSETS) - 1 - s] & (nb[:, s] >= 0)
    return torch.where(both, nb, -1)


def _tet(nx, ny, nz, seed):
    """Tetrahedron 6 c + p of box c is Kuhn's simplex of permutation p."""
    perms = list(itertools.permutations(range(3)))
    steps, dims = (1, nx, nx * ny), (nx, ny, nz)
    c = torch.arange(nx * ny * nz, device=DEV)
    at = (c % nx, (c // nx) % ny, c // (nx * ny))
    out = torch.empty((c.shape[0], 6, 4), dtype=torch.int64, device=DEV)
    for p, (a, b, d) in enumerate(perms):
        out[:, p, 0] = 6 * c + perms.index((b, a, d))
        out[:, p, 1] = 6 * c + perms.index((a, d, b))
        out[:, p, 2] = torch.where(at[a] + 1 < dims[a], 6 * (c + steps[a]) + perms.index((b, d, a)), -1)
        out[:, p, 3] = torch.where(at[d] > 0, 6 * (c - steps[d]) + perms.index((d, a, b)), -1)
    return out.reshape(-1, 4)


def _rcm(nb):
    """New index of every cell in reverse Cuthill-McKee order: breadth first,
    a level's cells by their first parent's place, then by degree."""
    n, slots = nb.shape
    deg = (nb >= 0).sum(1)
    place = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    first = torch.full((n,), 1 << 62, dtype=torch.int64, device=DEV)
    slot = torch.arange(slots, device=DEV)
    done = 0
    while done < n:
        level = torch.zeros(1, dtype=torch.int64, device=DEV) if done == 0 else torch.nonzero(place < 0)[:1, 0]
        while level.numel():
            place[level] = done + torch.arange(level.numel(), device=DEV)
            done += level.numel()
            child = nb[level]
            key = (torch.arange(level.numel(), device=DEV)[:, None] * 64 + deg[child.clamp(min=0)]) * slots + slot
            keep = (child >= 0) & (place[child.clamp(min=0)] < 0)
            child, key = child[keep], key[keep]
            first.scatter_reduce_(0, child, key, "amin")
            keep = first[child] == key
            child, key = child[keep], key[keep]
            level = child[torch.argsort(key)]
    return n - 1 - place


def _csr(mesh, nx, ny, nz, order, seed, long=0):
    """A scalar matrix as device tensors (row_ptr int32, col int32, val f64)."""
    nb = {"tet": _tet, "knn": _knn, "hex27": _hex27}[mesh](nx, ny, nz, seed)
    n = nb.shape[0]
    i = torch.arange(n, device=DEV)
    w = torch.stack([torch.where(nb[:, s] >= 0, 0.5 + _unit(_pair(i, nb[:, s].clamp(min=0), seed, 2)), 0.0)
                     for s in range(nb.shape[1])], 1)
    if order == "rcm":
        new = _rcm(nb)
    elif order == "random":
        new = torch.argsort(_mix(i + seed * 65537 + 3))
    else:
        new = i
    col = torch.cat([torch.where(nb >= 0, new[nb.clamp(min=0)], n), new[:, None]], 1)
    val = torch.cat([-w, w.sum(1, keepdim=True) + 1e-3], 1)
    del nb, w
    old = torch.empty_like(new)
    old[new] = i
    col, val = col[old], val[old]
    col, at = torch.sort(col, 1)
    val = torch.gather(val, 1, at)
    keep = col < n
    lens = keep.sum(1)
    col, val = col[keep], val[keep]
    if long:
        g = torch.Generator(device=DEV).manual_seed(seed + 99)
        where = torch.linspace(0, n - 1, long + 2, device=DEV, dtype=torch.float64)[1:-1].long().unique()
        size = max(1, n // 8)
        is_long = torch.zeros(n, dtype=torch.bool, device=DEV)
        is_long[where] = True
        stays = ~is_long.repeat_interleave(lens)
        row = torch.cat([i.repeat_interleave(lens)[stays], where.repeat_interleave(size)])
        extra = [torch.sort(torch.randperm(n, generator=g, device=DEV)[:size])[0] for _ in range(where.numel())]
        col = torch.cat([col[stays]] + extra)
        val = torch.cat([val[stays], 2 * torch.rand(size * where.numel(), generator=g, device=DEV, dtype=torch.float64) - 1])
        at = torch.argsort(row, stable=True)
        col, val = col[at], val[at]
        lens[where] = size
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(lens, 0)
    return ptr.to(torch.int32), col.to(torch.int32).contiguous(), val.contiguous()


def _blocks(nx, ny, nz, seed):
    """3x3 block CSR as device tensors, values (blocks, 3, 3)."""
    g = torch.Generator(device=DEV).manual_seed(seed + 7)
    n = nx * ny * nz
    i = torch.arange(n, device=DEV)
    faces = _lattice(nx, ny, nz, [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)])
    at = torch.stack([i % nx, (i // nx) % ny, i // (nx * ny)], 1)
    far = torch.randint(-2, 3, (n, 4, 3), generator=g, device=DEV) + at[:, None, :]
    dims = torch.tensor([nx, ny, nz], device=DEV)
    ok = ((far >= 0) & (far < dims)).all(2)
    ok &= torch.arange(4, device=DEV) < torch.randint(0, 5, (n, 1), generator=g, device=DEV)
    extra = torch.where(ok, far[..., 0] + nx * (far[..., 1] + ny * far[..., 2]), n)
    col = torch.sort(torch.cat([torch.where(faces >= 0, faces, n), extra], 1), 1)[0]
    col[:, 1:].masked_fill_(col[:, 1:] == col[:, :-1], n)
    keep = col < n
    lens = keep.sum(1)
    col = col[keep]
    val = 0.1 * torch.randn((col.numel(), 3, 3), generator=g, device=DEV, dtype=torch.float64)
    diag = col == i.repeat_interleave(lens)
    val[diag] += 4.0 * torch.eye(3, device=DEV, dtype=torch.float64)
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(lens, 0)
    return ptr.to(torch.int32), col.to(torch.int32), val


def _vector(shape, seed, dtype=torch.float64):
    g = torch.Generator(device=DEV).manual_seed(seed * 2 + 1)
    return (2 * torch.rand(shape, generator=g, device=DEV, dtype=torch.float64) - 1).to(dtype)


def _serving(case, seed):
    """The served matrices (host CSR) and the requests (matrix, vectors)."""
    r = np.random.default_rng(seed)
    mix = np.random.default_rng(case["largest"])  # who asks for what is the case's; the numbers are the seed's
    mats = []
    for m in range(case["matrices"]):
        edge = max(6, int(round(case["largest"] * (0.15 + 0.85 * (m + 1) / case["matrices"]))))
        p, c, v = _csr("hex27", edge, edge + 1, max(3, edge - 1), "rcm", seed + m)
        mats.append(SimpleNamespace(n_rows=p.numel() - 1, n_cols=p.numel() - 1, row_ptr=p.cpu().numpy(),
                                    col_idx=c.cpu().numpy(), values=v.cpu().numpy()))
    reqs = []
    for _ in range(case["requests"]):
        m = int(mix.integers(case["matrices"]))
        reqs.append((m, r.uniform(-1, 1, (int(mix.integers(1, case["most_k"] + 1)), mats[m].n_rows))))
    return mats, reqs


# ------------------------------------------------------------- the passes

def prepare(case, seed):
    if case["op"] == "serve":
        mats, reqs = _serving(case, seed)
        server = spmv.Server(hbm_budget_bytes=8 << 30, preload=True)
        ids = [server.add_matrix(A) for A in mats]
        server.drain()
        return SimpleNamespace(case=case, server=server, requests=[(ids[m], X) for m, X in reqs])
    dims = (case["nx"], case["ny"], case["nz"])
    if case["mesh"] == "block":
        p, c, v = _blocks(*dims, seed)
        n = p.numel() - 1
        M = spmv.Matrix.from_bsr3(n, n, p.cpu().numpy(), c.cpu().numpy(), v.cpu().numpy(), fp32=case["dtype"] == "f32")
        n *= 3
    else:
        p, c, v = _csr(case["mesh"], *dims, case["order"], seed, case.get("long", 0))
        n = p.numel() - 1
        kind = case.get("dtype") or case["mode"]
        torch.cuda.synchronize()  # the library copies the arrays on a stream of its own
        M = spmv.Matrix.from_device_csr(n, n, p, c, v, fp32=kind in ("f32", "f32v", "mixed"),
                                        bf16=kind in ("bf16", "pcg_bf16"))
    if case["op"] == "solve":
        return SimpleNamespace(case=case, M=M, b=_vector(n, seed))
    shape = n if case["k"] == 1 else (n, case["k"])
    X = _vector(shape, seed, VECTOR[case["dtype"]])
    return SimpleNamespace(case=case, M=M, X=X, Y=torch.empty_like(X))


def run(state):
    case = state.case
    if case["op"] == "serve":
        tickets = [state.server.submit_spmv(m, X) for m, X in state.requests]
        return [state.server.wait(t)[0] for t in tickets]
    if case["op"] == "solve":
        return state.M.cg(state.b, tol=case["tol"], mode=CG_MODES[case["mode"]])[0]
    if case["k"] > 1:
        return state.M.spmm_f32(state.X, state.Y) if case["dtype"] == "f32" else state.M.spmm(state.X, state.Y)
    product = {"f64": state.M.apply, "f32": state.M.apply_f32, "f32v": state.M.apply_f32v,
               "bf16": state.M.apply_bf16}[case["dtype"]]
    return product(state.X, state.Y)


def _entries(case, nx=None, ny=None, nz=None):
    """Rows and stored entries (blocks) of a case's mesh, in the mean over
    seeds (knn and block: 6.88 and 8.96 per row)."""
    nx, ny, nz = (nx, ny, nz) if nx else (case["nx"], case["ny"], case["nz"])
    n = nx * ny * nz
    if case["mesh"] == "tet":
        return 6 * n, 5 * 6 * n - 4 * (nx * ny + ny * nz + nx * nz)
    if case["mesh"] == "hex27":
        pairs = sum((nx - abs(a)) * (ny - abs(b)) * (nz - abs(c)) * (1.0 if abs(a) + abs(b) + abs(c) == 1 else 0.5)
                    for a, b, c in _OFFSETS)
        return n, int(n + pairs)
    if case["mesh"] == "block":
        return n, int(8.96 * n)
    k = case.get("long", 0)
    return n, int(6.88 * (n - k)) + k * (n // 8)


def work(case):
    if case["op"] == "serve":
        nbytes = flops = 0.0
        for m in range(case["matrices"]):
            e = max(6, int(round(case["largest"] * (0.15 + 0.85 * (m + 1) / case["matrices"]))))
            n, nnz = _entries(case, e, e + 1, max(3, e - 1))
            vectors = case["requests"] / case["matrices"] * (case["most_k"] + 1) / 2
            nbytes += 12 * nnz + 4 * n + vectors * 16 * n
            flops += vectors * 2 * nnz
        return {"bytes": nbytes, "flops": flops}
    n, nnz = _entries(case)
    if case["op"] == "solve":
        # iterations to 1e-10 grow slowly with the mesh (about 530 at 49K
        # cells, 1,200 at 16M); an iteration reads the matrix (its inner copy
        # in mixed precision) and makes nine vector passes
        its = 530 * (n / 49000) ** 0.14 * math.log(case["tol"]) / math.log(1e-10)
        vb, xb = (4, 4) if case["mode"] == "mixed" else (8, 8)
        return {"bytes": its * ((vb + 4) * nnz + 4 * n + 9 * xb * n), "flops": its * (2 * nnz + 10 * n)}
    vb, xb, k = VALUE_BYTES[case["dtype"]], VECTOR[case["dtype"]].itemsize, case["k"]
    if case["mesh"] == "block":
        return {"bytes": (9 * vb + 4) * nnz + 4 * n + 6 * k * xb * n, "flops": 18 * nnz * k}
    return {"bytes": (vb + 4) * nnz + 4 * n + 2 * k * xb * n, "flops": 2 * nnz * k}


# ------------------------------------------------------------ binary64

def _split(a):
    hi = (a * 134217729.0) - (a * 134217729.0 - a)
    return hi, a - hi


def _add_product(hi, lo, a, b):
    """(hi, lo) + a * b with the rounding errors of the product and of the
    sum kept in lo."""
    p = a * b
    (ah, al), (bh, bl) = _split(a), _split(b)
    e = ((ah * bh - p) + ah * bl + al * bh) + al * bl
    s = hi + p
    t = s - hi
    return s, lo + ((hi - (s - t)) + (p - t) + e)


def _times(ptr, col, val, X):
    """A X for a scalar matrix, X (n_cols, k)."""
    ptr, lens = ptr.long(), (ptr[1:] - ptr[:-1]).long()
    y = torch.zeros((ptr.numel() - 1, X.shape[1]), dtype=torch.float64, device=DEV)
    lo = torch.zeros_like(y)
    live = torch.arange(ptr.numel() - 1, device=DEV)
    j = 0
    while True:
        live = live[lens[live] > j]
        if live.numel() == 0:
            return y + lo
        if j >= 64:  # the few long rows: one at a time
            for r in live.tolist():
                a, b = int(ptr[r]) + j, int(ptr[r + 1])
                y[r] += (val[a:b, None] * X[col[a:b].long()]).sum(0)
            return y + lo
        at = ptr[live] + j
        a, b = val[at][:, None].expand(-1, X.shape[1]), X[col[at].long()]
        y[live], lo[live] = _add_product(y[live], lo[live], a, b)
        j += 1


def _solved(ptr, col, val, b):
    """x with A x = b by textbook CG (each row's entries padded to the
    longest), restarted from the true residual."""
    n = b.numel()
    lens = (ptr[1:] - ptr[:-1]).long()
    width = int(lens.max())
    slot = torch.arange(width, device=DEV)
    at = (ptr[:-1].long()[:, None] + slot).clamp(max=col.numel() - 1)
    inside = slot < lens[:, None]
    cols = torch.where(inside, col[at].long(), 0)
    vals = torch.where(inside, val[at], 0.0)
    del at, inside
    apply = lambda v: (vals * v[cols]).sum(1)  # noqa: E731
    x = torch.zeros_like(b)
    for _ in range(3):
        r = b - apply(x)
        p, rho, stop = r.clone(), r @ r, 1e-26 * (b @ b)
        for it in range(4000):
            q = apply(p)
            alpha = rho / (p @ q)
            x, r = x + alpha * p, r - alpha * q
            new = r @ r
            if it % 20 == 0 and float(new) < float(stop):
                break
            p, rho = r + (new / rho) * p, new
    assert x.numel() == n
    return x


def exact(case, seed):
    if case["op"] == "serve":
        mats, reqs = _serving(case, seed)
        dev = [[torch.as_tensor(a, device=DEV) for a in (A.row_ptr, A.col_idx, A.values)] for A in mats]
        return [_times(*dev[m], torch.as_tensor(X, device=DEV).T.contiguous()).T.contiguous() for m, X in reqs]
    dims = (case["nx"], case["ny"], case["nz"])
    if case["mesh"] == "block":
        p, c, v = _blocks(*dims, seed)
        n = p.numel() - 1
        if case["dtype"] == "f32":
            v = v.float().double()
        X = _vector(3 * n if case["k"] == 1 else (3 * n, case["k"]), seed, VECTOR[case["dtype"]]).double()
        Xb = X.reshape(n, 3 * case["k"])
        parts = []
        for r in range(3):  # scalar row r of every block row, column by column of the blocks
            cols = (3 * c.long()[:, None] + torch.arange(3, device=DEV)).reshape(-1)
            parts.append(_times(3 * p, cols, v[:, r, :].reshape(-1), Xb.reshape(3 * n, case["k"])))
        return torch.stack(parts, 1).reshape(X.shape)
    p, c, v = _csr(case["mesh"], *dims, case["order"], seed, case.get("long", 0))
    n = p.numel() - 1
    if case["op"] == "solve":
        return _solved(p, c, v, _vector(n, seed))
    if case["dtype"] in ("f32", "f32v"):
        v = v.float().double()
    elif case["dtype"] == "bf16":
        v = v.float().bfloat16().double()
    X = _vector(n if case["k"] == 1 else (n, case["k"]), seed, VECTOR[case["dtype"]]).double()
    return _times(p, c, v, X.reshape(n, -1)).reshape(X.shape)
