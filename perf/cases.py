"""What the performance of this framework is measured on: executions of the chain D = A (B C).

A case is one matrix A with a plan made once, as a solver, a graph network or a serving loop keeps it,
and one execution of the chain through the public entry points on operands that sit in device memory.
The matrices are those of the repository's benchmark configurations (tf_inputs.py): a band, the 5-point
and 7-point stencils in natural ordering and the symmetric R-MAT graph, made here on the GPU and at any
size.  B is dense ("gemm") or CSR ("spmm"); element types are fp32 and fp64; widths are the 32, 64 and
128 columns of the experiment grid and ragged ones (number of classes, number of right-hand sides).
Plans are made with the library's defaults: no tile parameters.
"""
import math

import torch

import paper_2407_00243_amd as tf


def _case(name, op, matrix, size, dtype, bcol, ccol, option="none", half_band=0, b_row=0):
    """size: rows (band, graph) or grid points along an edge (grid2d, grid3d).  bcol is 0 for a CSR B
    (square).  b_row: entries per row of a random CSR B, 0 = B is A itself.  option: "none",
    "transposed" (C handed over transposed), "static" (workspace of the library), "skip_unread"."""
    return {"name": name, "op": op, "matrix": matrix, "size": size, "half_band": half_band,
            "dtype": dtype, "bcol": bcol, "ccol": ccol, "b_row": b_row, "option": option}


def listed():
    return [
        # the smallest configuration: a band system with 32 right-hand sides; launches and latency
        _case("band_f64", "gemm", "band", 4096, "f64", 32, 32, half_band=8),
        # a serving loop that may not allocate: the entry point with the library's own workspace, on an
        # odd number of rows
        _case("band_f32_static", "gemm", "band", 20011, "f32", 64, 64, "static", half_band=5),
        # the 2D stencil configuration
        _case("grid2d_f32", "gemm", "grid2d", 512, "f32", 64, 64),
        # the same stencil at the wide double-precision end of the experiment grid
        _case("grid2d_f64_wide", "gemm", "grid2d", 512, "f64", 128, 128),
        # ragged widths on an odd grid: no row of B, C or D is 16-byte aligned
        _case("grid2d_f32_ragged", "gemm", "grid2d", 301, "f32", 50, 23),
        # one graph-convolution layer, forward, at the largest configuration's size
        _case("gcn_f32", "gemm", "graph", 1 << 20, "f32", 128, 128),
        # the last layer of a graph network: as many columns as there are classes
        _case("gcn_f32_classes", "gemm", "graph", 150000, "f32", 128, 41),
        # backward of a graph-convolution layer: A (G W^T), the weights handed over as they are stored
        _case("gcn_f32_backward", "gemm", "graph", 1 << 17, "f32", 64, 128, "transposed"),
        # A (A C) on the 3D stencil configuration: a block of vectors in a polynomial iteration
        _case("grid3d_f64", "spmm", "grid3d", 64, "f64", 0, 64),
        # the same in single precision on an odd grid with a ragged block of vectors
        _case("grid3d_f32_ragged", "spmm", "grid3d", 45, "f32", 0, 30),
        # two different irregular matrices: the largest CSR-B configuration
        _case("graph_f32", "spmm", "graph", 1 << 20, "f32", 0, 32, b_row=8),
        # the same kind in double precision, smaller and wider, rows of B C that nobody reads left out
        _case("graph_f64_skip", "spmm", "graph", 100003, "f64", 0, 64, "skip_unread", b_row=8),
    ]


def _rows(case):
    return case["size"] ** {"grid2d": 2, "grid3d": 3}.get(case["matrix"], 1)


def _entries(case):
    """Stored entries of A, to a few per cent for a graph."""
    n = _rows(case)
    return n * {"band": 2 * case["half_band"] + 1, "grid2d": 5, "grid3d": 7, "graph": 17}[case["matrix"]]


def _element(case):
    return 4 if case["dtype"] == "f32" else 8


def _cost(case):
    """Bytes that a plain execution asks for, dense operands and gathered rows."""
    n, w = _rows(case), case["ccol"] * _element(case)
    first = n * case["bcol"] * _element(case) if case["op"] == "gemm" else n * max(case["b_row"], 7) * w
    return first + _entries(case) * w + n * w


def draw(rng):
    largest = max(_cost(c) for c in listed())

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def width():
        return rng.choice([32, 64, 128]) if rng.random() < 0.5 else log_int(6, 128)

    op = rng.choice(["gemm", "gemm", "spmm"])
    matrix = rng.choice(["band", "grid2d", "grid3d", "graph", "graph"])
    size = {"band": lambda: log_int(3000, 400000), "grid2d": lambda: log_int(60, 720),
            "grid3d": lambda: log_int(15, 80), "graph": lambda: log_int(8000, 1 << 20)}[matrix]()
    option = "none"
    if op == "gemm":
        option = rng.choice(["none", "none", "transposed", "static"])
    elif matrix == "graph":
        option = rng.choice(["none", "skip_unread"])
    case = _case("", op, matrix, size, rng.choice(["f32", "f32", "f64"]), width() if op == "gemm" else 0,
                 width(), option, half_band=log_int(1, 24) if matrix == "band" else 0,
                 b_row=rng.randint(4, 12) if op == "spmm" and matrix == "graph" else 0)
    del case["name"]
    while _cost(case) > largest:
        case["size"] = int(case["size"] * 0.9)
    # the library's own workspace holds 64 MiB
    while option == "static" and _rows(case) * case["ccol"] * _element(case) > 60 << 20:
        case["size"] = int(case["size"] * 0.9)
    return case


# ------------------------------------------------------------------------------------ inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _uniform(gen, count, lo, hi, dtype):
    return torch.rand(count, generator=gen, device="cuda", dtype=dtype) * (hi - lo) + lo


def _graph_edges(n, gen):
    """Unique undirected edges lo < hi of a symmetric R-MAT graph (a, b, c, d = .57, .19, .19, .05) of
    average degree 16, without relabelling; draws that name a vertex beyond n are dropped."""
    bits = max(1, (n - 1).bit_length())
    draws = int(8 * n * ((1 << bits) / n) ** 0.6)
    src = torch.zeros(draws, dtype=torch.int64, device="cuda")
    dst = torch.zeros(draws, dtype=torch.int64, device="cuda")
    for _ in range(bits):
        u = torch.rand(draws, generator=gen, device="cuda")
        src = src * 2 + (u >= 0.76).to(torch.int64)
        dst = dst * 2 + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95)).to(torch.int64)
    keep = (src != dst) & (src < n) & (dst < n)
    src, dst = src[keep], dst[keep]
    key = torch.unique(torch.minimum(src, dst) * n + torch.maximum(src, dst))
    return key // n, key % n


def _csr(n, rows, cols, vals):
    order = torch.argsort(rows * n + cols)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return tf.DeviceCsr(n, n, rowptr.to(torch.int32), cols[order].to(torch.int32), vals[order].contiguous())


def _graph(case, gen, dtype):
    n = case["size"]
    lo, hi = _graph_edges(n, gen)
    if case["op"] == "gemm":
        # the propagation matrix of a graph network: D^-1/2 (Adj + I) D^-1/2
        diag = torch.arange(n, device="cuda")
        rows, cols = torch.cat([lo, hi, diag]), torch.cat([hi, lo, diag])
        deg = torch.bincount(rows, minlength=n).to(torch.float64)
        return _csr(n, rows, cols, (deg[rows] * deg[cols]).rsqrt().to(dtype))
    w = _uniform(gen, lo.numel(), 0.0, 1.0, dtype)
    return _csr(n, torch.cat([lo, hi]), torch.cat([hi, lo]), torch.cat([w, w]))


def _band(case, gen, dtype):
    n, h = case["size"], case["half_band"]
    rows = torch.arange(n, device="cuda").repeat_interleave(2 * h + 1)
    cols = rows + torch.arange(-h, h + 1, device="cuda").repeat(n)
    keep = (cols >= 0) & (cols < n)
    rows, cols = rows[keep], cols[keep]
    return _csr(n, rows, cols, _uniform(gen, rows.numel(), -1.0, 1.0, dtype))


def _grid(case, gen, dtype):
    """5- or 7-point stencil with varying coefficients, natural ordering, cut off at the boundary."""
    g, dims = case["size"], 2 if case["matrix"] == "grid2d" else 3
    n = g ** dims
    idx = torch.arange(n, device="cuda")
    rows, cols, vals = [idx], [idx], [_uniform(gen, n, 2.0 * dims, 3.0 * dims, dtype)]
    for d in range(dims):
        at = idx // g ** d % g
        for keep, step in ((at > 0, -g ** d), (at < g - 1, g ** d)):
            rows.append(idx[keep])
            cols.append(idx[keep] + step)
            vals.append(_uniform(gen, rows[-1].numel(), -1.5, -0.5, dtype))
    return _csr(n, torch.cat(rows), torch.cat(cols), torch.cat(vals))


def _random_rows(n, per_row, gen, dtype):
    """per_row uniform columns in every row, ascending, values U(-1, 1)."""
    cols = torch.randint(0, n, (n, per_row), generator=gen, device="cuda").sort(dim=1).values
    return tf.DeviceCsr(n, n, torch.arange(0, n * per_row + 1, per_row, device="cuda", dtype=torch.int32),
                        cols.reshape(-1).to(torch.int32), _uniform(gen, n * per_row, -1.0, 1.0, dtype))


def prepare(case, seed):
    gen = _generator(seed)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.float64
    n, ccol = _rows(case), case["ccol"]
    A = {"band": _band, "grid2d": _grid, "grid3d": _grid, "graph": _graph}[case["matrix"]](case, gen, dtype)
    flags = {"transposed": tf.TF_FLAG_C_TRANSPOSED, "skip_unread": tf.TF_FLAG_SKIP_UNREAD}.get(case["option"], 0)
    sparse = case["op"] == "spmm"
    bcol = n if sparse else case["bcol"]
    if sparse:
        B = _random_rows(n, case["b_row"], gen, dtype) if case["b_row"] else A
        C = torch.randn(n, ccol, generator=gen, device="cuda", dtype=dtype)
    else:
        B = torch.randn(n, bcol, generator=gen, device="cuda", dtype=dtype)
        shape = (ccol, bcol) if case["option"] == "transposed" else (bcol, ccol)
        C = torch.randn(*shape, generator=gen, device="cuda", dtype=dtype) / math.sqrt(bcol)
    return {"plan": tf.Plan(A, bcol, ccol, sparse, flags=flags), "static": case["option"] == "static",
            "B": B, "C": C, "D": torch.empty(n, ccol, device="cuda", dtype=dtype),
            "stream": torch.cuda.current_stream().cuda_stream}


def run(state):
    B, C, D, stream = state["B"], state["C"], state["D"], state["stream"]
    if state["static"]:
        tf.tf_gemm_spmm_static(state["plan"].handle, B, C, D, stream)
    else:
        state["plan"].run(B, C, D, stream)
    return D


def work(case):
    """A, B and C read once, D written once; the sparse product at the narrower of the two widths
    that the order of the two multiplications allows."""
    n, es, bcol, ccol = _rows(case), _element(case), case["bcol"], case["ccol"]
    nnz = _entries(case)
    if case["matrix"] == "graph":
        diag = n if case["op"] == "gemm" else 0
        nnz = 2 * _graph_edges(n, _generator(1))[0].numel() + diag
    a_bytes = 4 * (n + 1) + nnz * (4 + es)
    if case["op"] == "gemm":
        return {"bytes": a_bytes + (n * bcol + bcol * ccol + n * ccol) * es,
                "flops": 2 * n * bcol * ccol + 2 * nnz * min(bcol, ccol)}
    b_nnz = n * case["b_row"] or nnz
    b_bytes = 4 * (n + 1) + b_nnz * (4 + es) if case["b_row"] else 0
    return {"bytes": a_bytes + b_bytes + 2 * n * ccol * es, "flops": 2 * (b_nnz + nnz) * ccol}


def tolerance(case):
    # sums of products in the element type, in any order
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-13}
