"""What this library is timed on: its products, its solver loop and its server over the sizes they serve.

The matrices follow the laws of the repository's own generators (Zipf column lengths, a few
near-dense columns, uniform or Zipf-popular rows, lognormal values), drawn on the GPU from the seed.
Sizes: the benchmark's small, batching and large matrices, its document-term stand-in, and the ranges
of its served matrices (short side 500 .. 50,000, long side 50,000 .. 5,000,000, 1e5 .. 5e7 nonzeros,
1 .. 8 columns a request, blocks of up to 64 columns).  A program creates its matrix once and calls
products on it many times, so the created matrix is in the state and the calls are what is timed.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_1812_00904_amd import spw

STORAGE = {"f64": spw.SPW_F64, "f32": spw.SPW_F32, "bf16": spw.SPW_BF16}
VECTOR = {"f64": torch.float64, "f32": torch.float32}
VALUE_BYTES = {"f64": 8, "f32": 4, "bf16": 2}


def listed():
    def case(name, op, rows, cols, nnz, **more):
        # rows: short side, cols: long side; tall: the same arrays read by rows (CSR)
        c = {"name": name, "op": op, "rows": rows, "cols": cols, "nnz": nnz, "tall": False, "k": 1, "storage": "f64",
             "vector": "f64", "row_law": 0.0, "dense": 5, "dense_fill": 1.0, "lengths": "short", "transpose": False,
             "count": 0}
        c.update(more)
        return c

    return [
        # the smallest matrix of a served set, a request of three binary32 columns each way: launches and latency
        case("tiny tall k3", "pair", 500, 50_000, 100_000, tall=True, k=3, vector="f32"),
        # the benchmark's small matrix, one product each way, as a first-order method calls them: latency
        case("small wide", "pair", 1_000, 100_000, 1_000_000),
        # the document-term shape of the method's own experiments, one product each way
        case("documents", "pair", 19_996, 1_355_191, 9_100_000, row_law=0.5, dense=25, dense_fill=0.6, lengths="long"),
        # an ordinary tall matrix in binary32 throughout, odd sizes
        case("tall f32", "pair", 30_011, 2_000_003, 20_000_000, tall=True, storage="f32", vector="f32", row_law=0.8,
             dense=50, dense_fill=0.5),
        # bfloat16 values, binary32 vectors, the largest served shape
        case("wide bf16", "pair", 50_000, 5_000_000, 50_000_000, storage="bf16", vector="f32", row_law=0.8, dense=100,
             dense_fill=0.5),
        # the benchmark's headline matrix, one product each way: streaming from memory
        case("large wide", "pair", 50_000, 20_000_000, 200_000_000, row_law=0.8, dense=100, dense_fill=0.5),
        # a few right-hand sides on the batching matrix: A x for four columns at once
        case("batch Ax k4", "mv", 20_000, 5_000_000, 50_000_000, k=4, row_law=0.8, dense=100, dense_fill=0.5),
        # a served-size matrix with uniform rows and an odd block width, v^T A
        case("batch vA k7", "vtm", 5_003, 700_001, 7_000_000, k=7),
        # blocks of 16 in binary32 both ways, the transpose kept for them
        case("batch f32 k16", "pair", 20_000, 2_000_000, 20_000_000, k=16, storage="f32", vector="f32", row_law=0.8,
             dense=100, dense_fill=0.5, transpose=True),
        # the widest blocks on the batching matrix, both ways
        case("batch k64", "pair", 20_000, 5_000_000, 50_000_000, k=64, row_law=0.8, dense=100, dense_fill=0.5,
             transpose=True),
        # ten iterations of the least-squares solver: many short kernels one after another
        case("cgls", "cgls", 10_007, 500_000, 5_000_000, row_law=0.8, dense=20, dense_fill=0.5, count=10),
        # a burst of mixed requests on four resident matrices through the server
        case("serve burst", "serve", 3_000, 300_000, 2_000_000, count=24),
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))

    op = rng.choice(["pair", "pair", "pair", "pair", "mv", "vtm", "vtm", "cgls", "serve"])
    rows, cols = spread(500, 50_000), spread(50_000, 5_000_000)
    k = 1 if op in ("cgls", "serve") else rng.choice([1, 1, 1, spread(2, 8), spread(2, 8), spread(9, 64)])
    most = min(rows * cols // 2, 50_000_000, 1_000_000_000 // k, 10_000_000 if op in ("cgls", "serve") else 1 << 40)
    nnz = spread(100_000, max(most, 100_001))
    # values and vectors of one precision, or narrower values
    storage, vector = ("f64", "f64") if op in ("cgls", "serve") else rng.choice(
        [("f64", "f64"), ("f64", "f64"), ("f64", "f32"), ("f32", "f32"), ("bf16", "f32"), ("f32", "f64")])
    popular = rng.random() < 0.5
    return {"op": op, "rows": rows, "cols": cols, "nnz": nnz, "tall": rng.random() < 0.5, "k": k, "storage": storage,
            "vector": vector, "row_law": rng.choice([0.5, 0.8]) if popular else 0.0,
            "dense": rng.choice([0, 5, 25]), "dense_fill": rng.choice([0.5, 1.0]),
            "lengths": "long" if rng.random() < 0.25 else "short", "transpose": k >= 9 and rng.random() < 0.75,
            "count": {"cgls": rng.randint(3, 12), "serve": rng.randint(8, 32)}.get(op, 0)}


# ---------------------------------------------------------------- inputs

def _generator(seed, part):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 64 + part)


def _lengths(case, gen):
    """Column lengths: Zipf(1.1) on 1 .. K with the wanted mean, or a Zipf law fitted to a long tail."""
    rows, cols = case["rows"], case["cols"]
    dense = int(case["dense"] * case["dense_fill"] * rows)
    mean = max(case["nnz"] - dense, 0.2 * case["nnz"]) / cols
    if mean < 1.0:
        return (torch.rand(cols, generator=gen, device="cuda") < mean).long()
    ks = np.arange(1, max(rows // 2, 2) + 1, dtype=np.float64)
    if case["lengths"] == "long":
        lo, hi = 1.01, 4.0
        for _ in range(50):
            mid = 0.5 * (lo + hi)
            w = ks ** -mid
            lo, hi = (mid, hi) if (ks * w).sum() / w.sum() > mean else (lo, mid)
        w = ks ** -lo
    else:
        w = ks ** -1.1
        means = np.cumsum(w * ks) / np.cumsum(w)
        w = w[:min(int(np.searchsorted(means, mean)) + 1, w.size)]
    cdf = torch.from_numpy(np.cumsum(w) / w.sum()).cuda()
    u = torch.rand(cols, generator=gen, device="cuda", dtype=torch.float64)
    return torch.searchsorted(cdf, u).clamp_(max=w.size - 1) + 1


def _matrix(case, seed):
    """(ptr, row index, column index, value) of the short-by-long matrix in column order, on the GPU."""
    rows, cols = case["rows"], case["cols"]
    gen = _generator(seed, 1)
    lengths = _lengths(case, gen)
    total = int(lengths.sum())
    keys = torch.repeat_interleave(torch.arange(cols, device="cuda"), lengths, output_size=total) * rows
    if case["row_law"] > 0:
        w = torch.arange(1, rows + 1, device="cuda", dtype=torch.float64) ** -case["row_law"]
        cdf = torch.cumsum(w, 0) / w.sum()
        order = torch.randperm(rows, generator=gen, device="cuda")
        pick = torch.searchsorted(cdf, torch.rand(total, generator=gen, device="cuda", dtype=torch.float64))
        keys += order[pick.clamp_(max=rows - 1)]
        del pick
    else:
        keys += torch.randint(rows, (total,), generator=gen, device="cuda")
    if case["dense"]:
        at = torch.randint(cols, (case["dense"],), generator=gen, device="cuda")
        full = torch.rand((case["dense"], rows), generator=gen, device="cuda") < case["dense_fill"]
        which, row = full.nonzero(as_tuple=True)
        keys = torch.cat([keys, at[which] * rows + row])
    keys = torch.unique(keys)                       # sorted by column, then row; repeated entries dropped
    col = torch.div(keys, rows, rounding_mode="floor")
    row = (keys - col * rows).to(torch.int32)
    ptr = torch.zeros(cols + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.cumsum(torch.bincount(col, minlength=cols), 0)
    val = torch.randn(keys.numel(), generator=gen, device="cuda", dtype=torch.float64).exp_()
    val *= torch.randint(0, 2, (keys.numel(),), generator=gen, device="cuda") * 2 - 1
    return ptr, row, col, val


def _dense(n, k, dtype, gen):
    shape = (n,) if k == 1 else (n, k)
    return torch.rand(shape, generator=gen, device="cuda", dtype=VECTOR[dtype]) * 2 - 1


def _vectors(case, seed):
    """(input of A x, input of v^T A) for the matrix as its user sees it (m x n)."""
    m, n = _shape(case)
    gen = _generator(seed, 2)
    return _dense(n, case["k"], case["vector"], gen), _dense(m, case["k"], case["vector"], gen)


def _shape(case):
    return (case["cols"], case["rows"]) if case["tall"] else (case["rows"], case["cols"])


def _create(case, arrays):
    ptr, row, _, val = arrays
    m, n = _shape(case)
    opts = {"value_storage": STORAGE[case["storage"]]}
    if case["transpose"]:
        opts["transpose"] = 1
    return spw.SpwMatrix(spw.SPW_CSR if case["tall"] else spw.SPW_CSC, m, n, ptr.cpu().numpy(), row.cpu().numpy(),
                         val.cpu().numpy(), **opts)


def _requests(case):
    """The matrices of a served set (two wide, two tall, of different sizes) and a fixed mix of requests."""
    parts = []
    for i, scale in enumerate((1.0, 0.25, 0.5, 0.0625)):
        nnz = max(int(case["nnz"] * scale), 50_000)
        parts.append(dict(case, nnz=nnz, cols=max(int(case["cols"] * scale), 20_000), tall=i >= 2))
    mix = np.random.RandomState(7)
    wanted = [(int(mix.randint(4)), int(mix.randint(2)), int(mix.randint(1, 9)), "f32" if mix.rand() < 0.5 else "f64")
              for _ in range(case["count"])]
    return parts, wanted


class _Serving:
    """A server, its resident matrices and the blocks of every request; released in that order."""

    def __init__(self, case, seed):
        parts, self.wanted = _requests(case)
        self.matrices = [_create(p, _matrix(p, seed * 4 + i)) for i, p in enumerate(parts)]
        self.server = spw.Server()
        self.handles = [self.server.register(M) for M in self.matrices]
        self.blocks = []
        for i, (which, op, k, kind) in enumerate(self.wanted):
            m, n = _shape(parts[which])
            long_in, long_out = (n, m) if op == spw.SPW_OP_MV else (m, n)
            x = _dense(long_in, k, kind, _generator(seed, 3 + i))
            self.blocks.append((x, torch.zeros((long_out,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda")))
        torch.cuda.synchronize()                    # the server's streams read them

    def burst(self):
        tickets = [self.server.submit(self.handles[w[0]], w[1], x, y) for w, (x, y) in zip(self.wanted, self.blocks)]
        for t in tickets:
            self.server.wait(t)
        return [y for _, y in self.blocks]

    def __del__(self):
        self.server.close()
        for M in self.matrices:
            M.close()


def prepare(case, seed):
    if case["op"] == "serve":
        return {"case": case, "serving": _Serving(case, seed)}
    M = _create(case, _matrix(case, seed))
    x, v = _vectors(case, seed)
    m, n = _shape(case)
    if case["op"] == "cgls":
        return {"case": case, "M": M, "b": v, "x": torch.zeros(n, dtype=torch.float64, device="cuda")}
    return {"case": case, "M": M, "x": x, "v": v, "y": torch.zeros((m,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda"),
            "u": torch.zeros((n,) + tuple(v.shape[1:]), dtype=v.dtype, device="cuda")}


def run(state):
    op = state["case"]["op"]
    if op == "serve":
        return state["serving"].burst()
    M = state["M"]
    if op == "cgls":
        state["x"].zero_()                          # every solve starts from the same guess
        M.cgls(state["b"], state["x"], state["case"]["count"], hist=False)
        return state["x"]
    many = state["case"]["k"] > 1
    out = []
    if op in ("pair", "mv"):
        out.append((M.mv_batch if many else M.mv)(state["x"], state["y"]))
    if op in ("pair", "vtm"):
        out.append((M.vtm_batch if many else M.vtm)(state["v"], state["u"]))
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def _product_work(case, nnz, k, vector):
    sx = 8 if vector == "f64" else 4
    return (nnz * (VALUE_BYTES[case["storage"]] + 4) + 4 * (case["cols"] + 1) + k * (case["rows"] + case["cols"]) * sx,
            2 * nnz * k)


def work(case):
    if case["op"] == "serve":
        parts, wanted = _requests(case)
        each = [_product_work(parts[w[0]], parts[w[0]]["nnz"], w[2], w[3]) for w in wanted]
        return {"bytes": sum(e[0] for e in each), "flops": sum(e[1] for e in each)}
    b, f = _product_work(case, case["nnz"], case["k"], case["vector"])
    if case["op"] == "cgls":
        # two products an iteration and one for the start residual and gradient; p and x are read and written, s read
        return {"bytes": (case["count"] + 1) * 2 * b + case["count"] * 8 * (5 * _shape(case)[1]),
                "flops": (case["count"] + 1) * 2 * f}
    times = 2 if case["op"] == "pair" else 1
    return {"bytes": times * b, "flops": times * f}


# ---------------------------------------------------------------- the same results in 64 bits

def _stored(val, storage):
    if storage == "bf16":                           # to 8 significant bits at once, nearest, ties to even
        bits = val.view(torch.int64)
        return ((bits + ((1 << 44) - 1) + ((bits >> 45) & 1)) & -(1 << 45)).view(torch.float64)
    return val.float().double() if storage == "f32" else val


def _times(arrays, storage, x, out_len, out_is_row):
    """The product of the matrix (out_is_row) or its transpose with every column of x, in float64."""
    _, row, col, val = arrays
    to, of = (row, col) if out_is_row else (col, row)
    to, order = torch.sort(to, stable=True)         # the entries of each output, one after another
    of, val = of[order], _stored(val, storage)[order]
    lengths = torch.bincount(to, minlength=out_len)
    ends = torch.cumsum(lengths, 0)
    cols = x.double().reshape(x.shape[0], -1)
    out = torch.empty((out_len, cols.shape[1]), dtype=torch.float64, device="cuda")
    for c in range(cols.shape[1]):
        terms = val * cols[:, c].contiguous()[of]
        for a in range(0, out_len, 1 << 20):
            b = min(a + (1 << 20), out_len)
            first, last = int(ends[a] - lengths[a]), int(ends[b - 1])
            out[a:b, c] = torch.segment_reduce(terms[first:last], "sum", lengths=lengths[a:b], unsafe=True)
    return out.reshape((out_len,) + tuple(x.shape[1:]))


def _both(case, arrays):
    """(A x, v^T A) as functions of a vector or block, in float64."""
    m, n = _shape(case)
    return (lambda x: _times(arrays, case["storage"], x, m, not case["tall"]),
            lambda v: _times(arrays, case["storage"], v, n, case["tall"]))


def exact(case, seed):
    if case["op"] == "serve":
        parts, wanted = _requests(case)
        both = [_both(p, _matrix(p, seed * 4 + i)) for i, p in enumerate(parts)]
        out = []
        for i, (which, op, k, kind) in enumerate(wanted):
            m, n = _shape(parts[which])
            out.append(both[which][op](_dense(n if op == spw.SPW_OP_MV else m, k, kind, _generator(seed, 3 + i))))
        return out
    ax, va = _both(case, _matrix(case, seed))
    x, v = _vectors(case, seed)
    if case["op"] == "cgls":
        z = torch.zeros_like(x)
        r = v.clone()
        s = va(r)
        p, gamma = s.clone(), s @ s
        for _ in range(case["count"]):
            q = ax(p)
            alpha = gamma / (q @ q)
            z += alpha * p
            r -= alpha * q
            s = va(r)
            new = s @ s
            p = s + (new / gamma) * p
            gamma = new
        return z
    return ([ax(x)] if case["op"] in ("pair", "mv") else []) + ([va(v)] if case["op"] in ("pair", "vtm") else [])
