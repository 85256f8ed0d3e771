"""Performance cases: sparse times dense products as programs call them through the Python package.

A case is a dict of plain values:
  law    row-length law of A: "rmat" (power-law graph), "stencil" (27 points on a grid), "fixed", "poisson",
         "lognormal", "zipf" (the laws of ``workloads.sweep_csr``)
  rows, cols, mean   shape of A and its mean row length ("rmat": vertices, edge draws per vertex before duplicates
         merge; "stencil": rows = side ** 3)
  n      columns of the dense operand
  entry  how the program calls the library:
           "spmm"   ``DeviceCsr.spmm(X)``: statistics known, the rules choose the kernel
           "csr"    ``dgsp_spmm_csr`` with no statistics and no entry count, into a result the caller owns
           "axpby"  ``dgsp_spmm_csr_axpby``: Y = -A X + 0.5 Y, the update step of an iteration
           "slice"  ``dgsp_spmm_csr_ld``: X and Y are column slices of wider row-major matrices
           "train"  ``SparseOperator``: product and gradient with respect to X (the transposed product)
           "fresh"  a torch sparse CSR tensor that is new every time: statistics and one product

All inputs are made on the GPU from the seed alone: pattern, values and dense operand.
"""
import math

import torch

from paper_2106_16064_amd import binding as dgsp
from paper_2106_16064_amd.autograd import SparseOperator
from paper_2106_16064_amd.workloads import zipf_truncation

RMAT = (0.57, 0.19, 0.19, 0.05)
LAWS = ("rmat", "stencil", "fixed", "poisson", "lognormal", "zipf")
ENTRIES = ("spmm", "csr", "axpby", "slice", "train", "fresh")
ALPHA, BETA = -1.0, 0.5
SLICE_FROM = 5          # first column of the slice in the wider matrix
SLICE_EXTRA = 15        # columns of the wider matrix beyond the slice

# what no drawn case exceeds: entries and bytes of the largest listed cases, and multiplications short of the largest
# one's, because scattered columns cost more per multiplication than a power-law graph's
MOST_ENTRIES = 56_000_000
MOST_BYTES = 900_000_000
MOST_MULTIPLIES = 1_200_000_000


def _case(name, law, rows, mean, n, entry, cols=None):
    return dict(name=name, law=law, rows=rows, cols=cols or rows, mean=mean, n=n, entry=entry)


def listed():
    return [
        # a call so small that launches and host time are all of it (the smallest configuration of the benchmark)
        _case("tiny_poisson8_n4", "poisson", 4096, 8, 4, "spmm"),
        # graph analytics on a power-law graph: one SpMV per iteration (the headline configuration)
        _case("rmat20_n1", "rmat", 1 << 20, 16, 1, "spmm"),
        # feature aggregation of a graph network at its usual and its largest width
        _case("rmat20_n32", "rmat", 1 << 20, 16, 32, "spmm"),
        _case("rmat20_n128", "rmat", 1 << 20, 16, 128, "spmm"),
        # a PDE matrix: the SpMV of a solver and the product with a block of eight vectors
        _case("stencil128_n1", "stencil", 128 ** 3, 27, 1, "spmm"),
        _case("stencil128_n8", "stencil", 128 ** 3, 27, 8, "spmm"),
        # the update step of a solver on a mid-size grid with an odd side
        _case("stencil61_n1_axpby", "stencil", 61 ** 3, 27, 1, "axpby"),
        # training step of a graph network's last layer: product and gradient, as many columns as classes (odd)
        _case("rmat16_n41_train", "rmat", 1 << 16, 16, 41, "train"),
        # uneven rows through the call that knows nothing about the matrix
        _case("zipf16_n64_csr", "zipf", 1 << 18, 16, 64, "csr"),
        # long, equal rows with scattered columns, few vectors
        _case("fixed64_n4", "fixed", 1 << 18, 64, 4, "spmm"),
        # a rectangular operator on a column slice of wider matrices, odd sizes throughout
        _case("poisson12_n33_slice", "poisson", 100_003, 12, 33, "slice", cols=30_011),
        # sampled subgraphs: the matrix is new at every step
        _case("fresh_lognormal10_n32", "lognormal", 20_001, 10, 32, "fresh"),
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: law, size, mean row length and width over the listed ranges, all entries."""
    while True:
        law = rng.choice(LAWS)
        entry = rng.choice(ENTRIES)
        n = _log_between(rng, 1, 128)
        if law == "rmat":
            rows = 1 << rng.randint(12, 20)
            cols, mean = rows, _log_between(rng, 4, 32)
        elif law == "stencil":
            rows = _log_between(rng, 16, 128) ** 3
            cols, mean = rows, 27
        else:
            rows = _log_between(rng, 4096, 1 << 20)
            cols, mean = (_log_between(rng, 4096, 1 << 20) if rng.random() < 0.3 else rows), _log_between(rng, 4, 64)
        case = dict(law=law, rows=rows, cols=cols, mean=mean, n=n, entry=entry)
        times = 2 if entry == "train" else 1
        if rows * mean * times <= MOST_ENTRIES and rows * mean * n * times <= MOST_MULTIPLIES:
            if work(case)["bytes"] <= MOST_BYTES:
                return case


# ---------------------------------------------------------------------------------------------- matrices

def _rmat(rows, mean, gen):
    """Edges by quadrant choices, one level per bit; duplicates merged.  Values 1 / row length (mean aggregation)
    would make every row alike, so they are U(0, 1) as for weighted graphs."""
    scale = rows.bit_length() - 1
    edges = rows * mean
    a, b, c, _ = RMAT
    row = torch.zeros(edges, dtype=torch.int64, device="cuda")
    col = torch.zeros(edges, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        u = torch.rand(edges, device="cuda", generator=gen)
        row.mul_(2).add_(u >= a + b)
        col.mul_(2).add_(((u >= a) & (u < a + b)) | (u >= a + b + c))
    key = torch.unique(row.mul_(rows).add_(col))
    row = key // rows
    lens = torch.bincount(row, minlength=rows)
    return lens, (key - row * rows).to(torch.int32), torch.rand(key.numel(), device="cuda", generator=gen)


def _stencil(rows, gen):
    side = round(rows ** (1 / 3))
    at = torch.arange(rows, device="cuda", dtype=torch.int32)
    z, y, x = at // (side * side), at // side % side, at % side
    cols = torch.empty((rows, 27), dtype=torch.int32, device="cuda")
    inside = torch.empty((rows, 27), dtype=torch.bool, device="cuda")
    j = 0
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                zz, yy, xx = z + dz, y + dy, x + dx
                inside[:, j] = (zz >= 0) & (zz < side) & (yy >= 0) & (yy < side) & (xx >= 0) & (xx < side)
                cols[:, j] = (zz * side + yy) * side + xx
                j += 1
    vals = torch.randn((rows, 27), device="cuda", generator=gen)
    vals[:, 13] += 27.0
    return inside.sum(1), cols[inside], vals[inside]


def _random_columns(lens, cols, gen):
    """Distinct uniform columns per row, ascending: drawn with replacement, collisions drawn again."""
    rows = torch.repeat_interleave(torch.arange(lens.numel(), device="cuda"), lens)
    key = rows * cols + torch.randint(0, cols, (rows.numel(),), device="cuda", generator=gen)
    while True:
        key = torch.sort(key).values
        again = torch.zeros_like(key, dtype=torch.bool)
        again[1:] = key[1:] == key[:-1]
        count = int(again.sum())
        if count == 0:
            return (key - rows * cols).to(torch.int32)
        key[again] = rows[again] * cols + torch.randint(0, cols, (count,), device="cuda", generator=gen)


def _lengths(case, gen):
    rows, mean = case["rows"], float(case["mean"])
    if case["law"] == "fixed":
        lens = torch.full((rows,), mean, device="cuda")
    elif case["law"] == "poisson":
        lens = torch.poisson(torch.full((rows,), mean, device="cuda"), generator=gen)
    elif case["law"] == "lognormal":
        lens = torch.round(torch.exp(torch.randn(rows, device="cuda", generator=gen) + (math.log(mean) - 0.5)))
    else:
        most = zipf_truncation(mean)
        cdf = torch.cumsum(torch.arange(1, most + 1, dtype=torch.float64, device="cuda") ** -1.5, 0)
        u = torch.rand(rows, dtype=torch.float64, device="cuda", generator=gen)
        lens = torch.searchsorted(cdf / cdf[-1], u).add_(1).clamp_(max=most)
    return lens.to(torch.int64).clamp_(0, case["cols"] // 4)


def _matrix(case, gen):
    if case["law"] == "rmat":
        lens, colidx, vals = _rmat(case["rows"], case["mean"], gen)
    elif case["law"] == "stencil":
        lens, colidx, vals = _stencil(case["rows"], gen)
    else:
        lens = _lengths(case, gen)
        colidx = _random_columns(lens, case["cols"], gen)
        vals = torch.rand(colidx.numel(), device="cuda", generator=gen) * 2 - 1
    rowptr = torch.zeros(case["rows"] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=rowptr[1:])
    return rowptr, colidx, vals


# ---------------------------------------------------------------------------------------------- what is measured

def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    M, K, n, entry = case["rows"], case["cols"], case["n"], case["entry"]
    rowptr, colidx, vals = _matrix(case, gen)
    s = dict(entry=entry, M=M, K=K, n=n)
    X = torch.randn((K, n), device="cuda", generator=gen)
    if entry == "fresh":
        s["T"] = torch.sparse_csr_tensor(rowptr, colidx.to(torch.int64), vals, size=(M, K))
        s["X"] = X
        return s
    A = s["A"] = dgsp.DeviceCsr.from_device(M, K, rowptr, colidx, vals)
    s["X"] = X
    if entry == "csr":
        s["Y"] = torch.empty((M, n), device="cuda")
    elif entry == "axpby":
        s["Y"] = torch.randn((M, n), device="cuda", generator=gen)
    elif entry == "slice":
        wide = n + SLICE_EXTRA
        s["X"] = torch.randn((K, wide), device="cuda", generator=gen)[:, SLICE_FROM:SLICE_FROM + n]
        s["Y"] = torch.zeros((M, wide), device="cuda")[:, SLICE_FROM:SLICE_FROM + n]
    elif entry == "train":
        s["op"] = SparseOperator(A)
        s["X"].requires_grad_(True)
        s["dY"] = torch.randn((M, n), device="cuda", generator=gen)
    return s


def run(s):
    entry = s["entry"]
    if entry == "spmm":
        return s["A"].spmm(s["X"])
    if entry == "fresh":
        return dgsp.DeviceCsr.from_torch_sparse_csr(s["T"]).spmm(s["X"])
    if entry == "train":
        X = s["X"]
        X.grad = None
        Y = s["op"](X)
        Y.backward(s["dY"])
        return {"y": Y.detach(), "dx": X.grad}
    A, X, Y = s["A"], s["X"], s["Y"]
    if entry == "csr":
        dgsp.dgsp_spmm_csr(s["M"], s["K"], s["n"], A.rowptr, A.colidx, A.vals, X, Y, dgsp.AUTO)
    elif entry == "axpby":
        dgsp.dgsp_spmm_csr_axpby(s["M"], s["K"], s["n"], A.nnz, A.rowptr, A.colidx, A.vals, X, Y, ALPHA, BETA,
                                 features=A.features)
    else:
        dgsp.dgsp_spmm_csr_ld(s["M"], s["K"], s["n"], A.nnz, A.rowptr, A.colidx, A.vals, X, Y, features=A.features)
    return Y


# ---------------------------------------------------------------------------------------------- what it costs at least

def _expected(case):
    """Expected stored entries, columns that hold one, rows that hold one."""
    rows, cols, mean = case["rows"], case["cols"], float(case["mean"])
    if case["law"] == "stencil":
        side = round(rows ** (1 / 3))
        return float((3 * side - 2) ** 3), rows, rows
    if case["law"] == "rmat":
        scale, edges = rows.bit_length() - 1, rows * case["mean"]
        a, b, c, d = RMAT
        hit = lambda p: -math.expm1(edges * math.log1p(-p))  # noqa: E731  (an event of probability p in any draw)
        f = math.factorial
        nnz = 0.0
        for i in range(scale + 1):
            for j in range(scale + 1 - i):
                for k in range(scale + 1 - i - j):
                    m = scale - i - j - k
                    nnz += f(scale) // (f(i) * f(j) * f(k) * f(m)) * hit(a ** i * b ** j * c ** k * d ** m)
        used = sum(math.comb(scale, k) * hit((a + c) ** (scale - k) * (b + d) ** k) for k in range(scale + 1))
        return nnz, used, used        # rows and columns follow the same law (b == c)
    nnz = rows * mean
    return nnz, cols * -math.expm1(nnz * math.log1p(-1.0 / cols)), rows


def work(case):
    nnz, used_cols, used_rows = _expected(case)
    M, K, n, entry = case["rows"], case["cols"], case["n"], case["entry"]
    index, pointer = (8, 8) if entry == "fresh" else (4, 4)
    moved = (index + 4) * nnz + pointer * (M + 1) + 4 * n * (used_cols + M)
    if entry == "axpby":
        moved += 4 * n * M                                                  # the old Y
    if entry == "train":
        moved += 8 * nnz + 4 * (K + 1) + 4 * n * (used_rows + K)            # the transposed product
    return {"bytes": moved, "flops": 2 * nnz * n * (2 if entry == "train" else 1)}


def tolerance(case):
    """32-bit products and sums in any order, rows up to tens of thousands of entries."""
    return {"rel": 1e-5, "max": 1e-4}
