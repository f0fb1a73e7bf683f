"""The work that users of this library have it do, as measurable cases.

Three kinds of call, each through the Python binding:

* ``product``: one ``H2Operator.gemv`` -- the H^2 matrix-vector or
  multi-vector product, op 'N' or 'T', FP64 or with the low-rank data in FP32
  or BF16;
* ``batch``: one ``H2Batch.gemv`` over many independent operators;
* ``compress``: one ``H2Operator.compress`` and a product with the new
  operator.

A program loads an operator once and multiplies with it many times, so the
loaded (and, where the case says so, tuned) handle is kept from one
``prepare`` to the next; the vectors are new for every seed.  Operators are
kernel matrices on uniform random points, from the seeded generator that the
benchmark uses.
"""
import math
import random

import numpy as np
import torch

import h2gen
from paper_2109_05451_amd import H2Batch, H2Operator

_LEAF, _ETA = 64, 0.7


def _product(name, n, dim=2, leaf=_LEAF, p=6, kernel="exp", param=0.1, op="N", prec="fp64", nv=1, alpha=1.0,
             beta=0.0, tune=False):
    c = dict(kind="product", n=n, dim=dim, leaf=leaf, p=p, eta=_ETA, kernel=kernel, param=param, op=op, prec=prec,
             nv=nv, alpha=alpha, beta=beta, tune=tune)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one product with a small operator inside an iterative solver: the
        # call is a chain of dependent launches, its latency is what counts
        _product("small_nv1", 4096, p=4),
        # the headline product of the benchmark: one GPU's share of a 2D
        # kernel operator, one vector
        _product("large_nv1", 1 << 20),
        # the same operator in a block Krylov method (16 vectors) and in
        # randomized sampling (64 vectors), tuned once as the benchmark does
        _product("large_nv16", 1 << 20, nv=16, tune=True),
        _product("large_nv64", 1 << 20, nv=64, tune=True),
        # a residual update on a mid-sized operator straight after loading:
        # odd point count, odd rank (25), ragged leaves, odd vector count
        _product("ragged_nv7", 100003, leaf=50, p=5, kernel="gauss", param=0.15, nv=7, alpha=1.5, beta=-0.5),
        # the adjoint product: one vector (least squares, adjoint solves) and
        # a block (the transposed pass of randomized sampling)
        _product("transpose_nv1", 1 << 18, op="T"),
        _product("transpose_nv24", 100003, leaf=50, p=5, op="T", nv=24),
        # 3D Green's function of the Laplacian, rank 64, 64 vectors, FP64 and
        # with BF16 low-rank data
        _product("volume_nv64", 1 << 17, dim=3, p=4, kernel="laplace", param=0.0, nv=64, tune=True),
        _product("volume_nv64_bf16", 1 << 17, dim=3, p=4, kernel="laplace", param=0.0, nv=64, prec="bf16", tune=True),
        # FP32 low-rank data, a block of 16 vectors, untuned
        _product("mixed_nv16_fp32", 1 << 18, nv=16, prec="fp32"),
        # many small independent operators in one call, each with its own
        # vector count in 1..32
        dict(name="batch_48", kind="batch", count=48, base=3000, nmin=12.0, nmax=16.0),
        # recompression after a high-accuracy construction, and the first
        # product with the compressed operator
        dict(name="compress_64k", kind="compress", n=1 << 16, leaf=_LEAF, p=6, eta=0.9, tau=1e-3, nv=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.random()
    if kind < 0.08:
        return dict(kind="batch", count=rng.randint(4, 40), base=rng.randrange(10000, 90000), nmin=11.0, nmax=15.5)
    if kind < 0.14:
        return dict(kind="compress", n=_log_int(rng, 3000, 1 << 16), leaf=rng.randint(40, 64),
                    p=rng.choice([4, 5, 6]), eta=0.9, tau=rng.choice([1e-2, 1e-3, 1e-4]), nv=rng.randint(1, 8))
    dim = 3 if rng.random() < 0.25 else 2
    n = _log_int(rng, 1000, 100000 if dim == 3 else 1 << 20)
    leaf = rng.randint(32, 64) if n < 1 << 18 else rng.randint(56, 64)
    p = rng.choice([3, 4]) if dim == 3 else rng.choice([4, 5, 6])
    kernel = "laplace" if dim == 3 else rng.choice(["exp", "gauss"])
    prec = rng.choice(["fp64", "fp64", "fp64", "fp32", "bf16"])
    op = "T" if prec != "bf16" and rng.random() < 0.3 else "N"
    nv = _log_int(rng, 1, 64)
    beta = rng.choice([0.0, 0.0, 0.5, -0.25])
    return _product(None, n, dim, leaf, p, kernel, 0.0 if dim == 3 else round(rng.uniform(0.05, 0.2), 3), op, prec,
                    nv, rng.choice([1.0, 1.5, -1.0]), beta, tune=rng.random() < 0.25)


# ---- operators


def _spec(case):
    """The construction of a case's operator (points, tree, kernel)."""
    if case["kind"] == "compress":
        return (case["n"], 2, case["leaf"], case["p"], case["eta"], "exp", 0.1)
    return tuple(case[k] for k in ("n", "dim", "leaf", "p", "eta", "kernel", "param"))


def _batch_specs(case):
    """(construction, vectors) of every operator of a batch: sizes, leaves,
    ranks, kernel widths and vector counts of the benchmark's batch."""
    out = []
    for i in range(case["count"]):
        r = random.Random(case["base"] + i)
        n = int(round(2 ** r.uniform(case["nmin"], case["nmax"])))
        out.append(((n, 2, r.randint(32, 64), r.choice([4, 5, 6]), _ETA, "exp", round(r.uniform(0.05, 0.2), 3)),
                    r.randint(1, 32)))
    return out


def _build(spec):
    n, dim, leaf, p, eta, kernel, param = spec
    return h2gen.build(h2gen.points(n, dim, 1000 + n + dim), leaf, p, eta, kernel, param)


_KEEP_BYTES = 120 << 30  # device memory of the handles kept between preparations
_handles = {}            # key -> [handle, what it is tuned for, device bytes]
_sizes = {}              # operator construction -> stored entries


def _evict(need):
    while _handles and sum(h[2] for h in _handles.values()) + need > _KEEP_BYTES:
        _handles.pop(next(iter(_handles)))[0].close()


def _operator(spec):
    if spec not in _handles:
        buf = _build(spec)
        _sizes[spec] = _entries(buf.array)
        _evict(4 * buf.nbytes)
        _handles[spec] = [H2Operator(buf.array), None, 4 * buf.nbytes]
        buf.free()
    return _handles[spec]


def _columns(n, nv, gen):
    return torch.randn(nv, n, dtype=torch.float64, device="cuda", generator=gen).t()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "batch":
        specs = _batch_specs(case)
        nvs = [nv for _, nv in specs]
        Xs = [_columns(s[0], nv, gen) for s, nv in specs]
        Ys = [torch.empty((nv, s[0]), dtype=torch.float64, device="cuda").t() for s, nv in specs]
        key = ("batch", case["count"], case["base"], case["nmin"], case["nmax"])
        if key not in _handles:
            bufs = [_build(s) for s, _ in specs]
            for (s, _), b in zip(specs, bufs):
                _sizes[s] = _entries(b.array)
            size = 4 * sum(b.nbytes for b in bufs)
            _evict(size)
            _handles[key] = [H2Batch([b.array for b in bufs], nv_max=nvs), None, size]
            _handles[key][0].tune(Xs, Ys)
            for b in bufs:
                b.free()
        return {"case": case, "A": _handles[key][0], "X": Xs, "Y": Ys}
    held = _operator(_spec(case))
    A = held[0]
    state = {"case": case, "A": A, "X": _columns(case["n"], case["nv"], gen), "Y": None}
    if case["kind"] == "product":
        A.prepare(case["prec"])
        A.reserve(case["nv"])
        if case["tune"] and held[1] != (case["nv"], case["prec"]):
            A.tune(case["nv"], case["prec"])
            held[1] = (case["nv"], case["prec"])
        if case["beta"] != 0.0:
            state["Y"] = _columns(case["n"], case["nv"], gen)
    return state


def run(state):
    case, A = state["case"], state["A"]
    if case["kind"] == "batch":
        A.gemv(state["X"], state["Y"])
        return state["Y"]
    if case["kind"] == "compress":
        C, _ = A.compress(case["tau"])
        Y = C.gemv(state["X"])
        ranks, _ = C.ranks()
        C.close()
        return {"Y": Y, "ranks": ranks}
    return A.gemv(state["X"], op=case["op"], alpha=case["alpha"], beta=case["beta"], Y=state["Y"],
                  precision=case["prec"])


# ---- the representation's arrays and the work of a pass


def _arrays(b):
    """Numpy views of a serialized representation (little-endian 8-byte
    elements, sections on 64-byte boundaries, matrices column-major)."""
    flags = int(b[12:16].view(np.uint32)[0])
    n, q, nnodes, dim = (int(x) for x in b[16:48].view(np.int64))
    pos = 128

    def take(count, dt):
        nonlocal pos
        pos = (pos + 63) // 64 * 64
        a = b[pos:pos + 8 * count].view(dt)
        pos += 8 * count
        return a

    i64, f64 = np.int64, np.float64
    ndense = int(b[88:96].view(i64)[0])
    r = {"n": n, "q": q}
    lp = r["lp"] = take(q + 2, i64)
    kr, kc, nadm = take(q + 1, i64), take(q + 1, i64), take(q + 1, i64)
    r["perm"], lo, hi, r["parent"] = take(n, i64), take(nnodes, i64), take(nnodes, i64), take(nnodes, i64)
    rp, col = take(nnodes + q + 1, i64), take(int(nadm.sum()), i64)
    r["rp"] = [rp[lp[l] + l:lp[l + 1] + l + 1] for l in range(q + 1)]
    cb = np.concatenate([[0], np.cumsum(nadm)])
    r["col"] = [col[cb[l]:cb[l + 1]] for l in range(q + 1)]
    r["drp"], r["dcol"] = take(int(lp[q + 1] - lp[q]) + 1, i64), take(ndense, i64)
    nodes = np.diff(lp)
    sep = flags & 1
    r["kr"], r["kc"] = kr, kc
    ne = int(sum(nodes[l] * kr[l] * kr[l - 1] for l in range(1, q + 1)))
    nf = int(sum(nodes[l] * kc[l] * kc[l - 1] for l in range(1, q + 1)))
    r["U"], r["E"] = take(n * int(kr[q]), f64), take(ne, f64)
    r["V"], r["F"] = take(n * int(kc[q]) if sep else 0, f64), take(nf if sep else 0, f64)
    r["S"] = take(int((nadm * kr * kc).sum()), f64)
    r["lo"], r["m"] = lo[lp[q]:], (hi - lo)[lp[q]:]
    t = np.repeat(np.arange(len(r["m"])), np.diff(r["drp"]))
    r["dt"] = t
    r["dsz"] = r["m"][t] * r["m"][r["dcol"]]
    r["D"] = take(int(r["dsz"].sum()), f64)
    return r


def _entries(b):
    r = _arrays(b)
    return {"lowrank": sum(r[k].size for k in "UEVFS"), "dense": r["D"].size,
            # entries read by a product: a shared basis serves both sweeps
            "used": sum(r[k].size for k in "UEVFS") + (r["U"].size + r["E"].size if not r["V"].size else 0)}


def _size_of(spec):
    if spec not in _sizes:
        buf = _build(spec)
        _sizes[spec] = _entries(buf.array)
        buf.free()
    return _sizes[spec]


def work(case):
    """Stored data read once (low-rank part at its precision, dense blocks and
    vectors in FP64), X read and Y written once (and read where beta != 0);
    two flops per used entry and vector.  A recompression reads the stored
    data and writes the dense blocks and the (much smaller) new low-rank part;
    its flops are counted as those of the product that follows."""
    if case["kind"] == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for spec, nv in _batch_specs(case):
            e = _size_of(spec)
            total["bytes"] += 8.0 * (e["lowrank"] + e["dense"] + 2 * spec[0] * nv)
            total["flops"] += 2.0 * nv * (e["used"] + e["dense"])
        return total
    e, n, nv = _size_of(_spec(case)), case["n"], case["nv"]
    if case["kind"] == "compress":
        return {"bytes": 8.0 * (e["lowrank"] + 3 * e["dense"] + 2 * n * nv), "flops": 2.0 * nv * e["dense"]}
    width = {"fp64": 8, "fp32": 4, "bf16": 2}[case["prec"]]
    vectors = 8.0 * n * nv * (2 + (case["beta"] != 0.0))
    return {"bytes": width * e["lowrank"] + 8.0 * e["dense"] + vectors, "flops": 2.0 * nv * (e["used"] + e["dense"])}


# ---- the product in 64 bits, from its definition


def _blocks(D, off, rows, cols):
    """len(off) column-major rows x cols blocks of the flat array D."""
    ix = off[:, None] + torch.arange(rows * cols, device=D.device)
    return D[ix].view(-1, cols, rows).transpose(1, 2)


def _multiply(r, X, trans):
    """op(A) X in original order: leaf products, transfers up, coupling
    blocks, transfers down, leaf expansion, dense blocks."""
    dev = X.device
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    q, lp, nv = r["q"], r["lp"], X.shape[1]
    U, E = to(r["U"]), to(r["E"])
    V, F = (to(r["V"]), to(r["F"])) if r["V"].size else (U, E)
    kr, kc = [int(k) for k in r["kr"]], [int(k) for k in r["kc"]]
    if trans:
        U, E, V, F, kr, kc = V, F, U, E, kc, kr
    perm, parent = to(r["perm"]), to(r["parent"])
    lo, m = to(r["lo"]), to(r["m"])
    x = X[perm].contiguous()
    y = torch.zeros_like(x)
    sizes = [int(s) for s in torch.unique(m) if s > 0]
    at = lambda ts, s: lo[ts][:, None] + torch.arange(s, device=dev)  # noqa: E731
    step = max(1, (1 << 28) // (64 * 64 * 8))
    # up
    xh = [None] * (q + 1)
    xh[q] = torch.zeros(len(m), kc[q], nv, dtype=torch.float64, device=dev)
    for s in sizes:
        for ts in torch.nonzero(m == s).flatten().split(step):
            xh[q][ts] = torch.bmm(_blocks(V, lo[ts] * kc[q], s, kc[q]).transpose(1, 2).contiguous(), x[at(ts, s)])
    transfer = lambda A, off, count, a, b: A[off:off + count * a * b].view(count, b, a).transpose(1, 2)  # noqa: E731
    eo, fo = [0] * (q + 2), [0] * (q + 2)
    for l in range(1, q + 1):
        c = int(lp[l + 1] - lp[l])
        eo[l + 1], fo[l + 1] = eo[l] + c * kr[l] * kr[l - 1], fo[l] + c * kc[l] * kc[l - 1]
    for l in range(q, 0, -1):
        c, up = int(lp[l + 1] - lp[l]), int(lp[l] - lp[l - 1])
        Ft = transfer(F, fo[l], c, kc[l], kc[l - 1]).transpose(1, 2).contiguous()
        xh[l - 1] = torch.zeros(up, kc[l - 1], nv, dtype=torch.float64, device=dev)
        xh[l - 1].index_add_(0, parent[lp[l]:lp[l + 1]] - int(lp[l - 1]), torch.bmm(Ft, xh[l]))
    # coupling, then down
    yh, so = None, 0
    for l in range(q + 1):
        c = int(lp[l + 1] - lp[l])
        cur = torch.zeros(c, kr[l], nv, dtype=torch.float64, device=dev)
        rows = to(np.repeat(np.arange(c), np.diff(r["rp"][l])))
        cols = to(r["col"][l])
        a, b = (kc[l], kr[l]) if trans else (kr[l], kc[l])
        nb = len(cols)
        for i in range(0, nb, step):
            j = min(nb, i + step)
            S = to(r["S"][so + i * a * b:so + j * a * b]).view(j - i, b, a)
            S = S if trans else S.transpose(1, 2).contiguous()
            src, dst = (rows, cols) if trans else (cols, rows)
            cur.index_add_(0, dst[i:j], torch.bmm(S, xh[l][src[i:j]]))
        so += nb * a * b
        if l > 0:
            cur += torch.bmm(transfer(E, eo[l], c, kr[l], kr[l - 1]).contiguous(),
                             yh[parent[lp[l]:lp[l + 1]] - int(lp[l - 1])])
        yh = cur
    for s in sizes:
        for ts in torch.nonzero(m == s).flatten().split(step):
            y[at(ts, s)] += torch.bmm(_blocks(U, lo[ts] * kr[q], s, kr[q]).contiguous(), yh[ts])
    # dense blocks, by shape
    doff = np.concatenate([[0], np.cumsum(r["dsz"])])
    for i in range(0, len(r["dt"]), step):
        j = min(len(r["dt"]), i + step)
        D = to(r["D"][doff[i]:doff[j]])
        off, dt, ds = to(doff[i:j] - doff[i]), to(r["dt"][i:j]), to(r["dcol"][i:j])
        for a in sizes:
            for b in sizes:
                w = torch.nonzero((m[dt] == a) & (m[ds] == b)).flatten()
                if not len(w):
                    continue
                B = _blocks(D, off[w], a, b)
                B = (B.transpose(1, 2) if trans else B).contiguous()
                src, dst = (dt, ds) if trans else (ds, dt)
                sa, sb = (b, a) if trans else (a, b)
                y.view(-1, nv).index_add_(0, at(dst[w], sa).flatten(),
                                          torch.bmm(B, x[at(src[w], sb)]).reshape(-1, nv))
    out = torch.empty_like(y)
    out[perm] = y
    return out


_last = [None, None]  # the operator last parsed for exact()


def _exact_product(spec, X, op="N"):
    if _last[0] != spec:
        _last[:] = [None, None]
        buf = _build(spec)
        _last[:] = [spec, (buf, _arrays(buf.array))]
    return _multiply(_last[1][1], X, op == "T")


def exact(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "batch":
        specs = _batch_specs(case)
        Xs = [_columns(s[0], nv, gen) for s, nv in specs]
        return [_exact_product(s, X) for (s, _), X in zip(specs, Xs)]
    if case["kind"] == "compress":
        return None  # which directions are kept is the algorithm's own choice
    X = _columns(case["n"], case["nv"], gen)
    Y = case["alpha"] * _exact_product(_spec(case), X, case["op"])
    if case["beta"] != 0.0:
        Y += case["beta"] * _columns(case["n"], case["nv"], gen)
    return Y
