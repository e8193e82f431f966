"""The work this library is used for, as measurable cases: what a program has in hand before a call (``prepare``),
one pass through the public entry points (``run``), and what that pass cannot do without (``work``).

Operations
  spmm       C = A @ B on a converted matrix with its own values
  step       SDDMM into the value array, then SpMM, through the closures of ``bind_sddmm`` / ``bind_spmm``
             (a loop that repeats one call)
  attention  softmax_rows(scale * X Y^T at A's pattern) @ H, the inference pass of a graph attention layer
  train      forward and backward of that layer: SDDMM, edge softmax, SpMM, and the gradients of X, Y and H
             through the second format, that of A^T
  scores     SDDMM in CSR order: link scores, or the gradient of A's values
  reweight   new edge weights in CSR order carried into the format, then SpMM (weights that change per step)
  convert    CSR -> window format, the once-per-pattern preparation
  transpose  CSR of A^T and A's values in its order

Patterns (the synthetic families of ``workloads/``): ``uniform`` (about ``deg`` entries per row at uniformly random
columns, any M x K), ``rmat`` (power-law graph, a/b/c/d = .57/.19/.19/.05), ``stencil`` (5-point stencil on a
grid), ``lognormal`` (row degrees exp(N(2.5, 1)), columns uniform).  Duplicate draws are stored once.
"""
import math

import torch

import paper_2412_11007_amd as fs

RMAT = (0.57, 0.19, 0.19, 0.05)


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: a few thousand rows, where launches and the host path count
        dict(name="spmm_uniform_4k", op="spmm", pattern="uniform", M=4096, K=4096, deg=16, N=32, dtype="f16"),
        # attention over a small graph or one sampled neighbourhood, one head
        dict(name="attention_rmat13", op="attention", pattern="rmat", scale=13, edge_factor=16, d=32, N=64, dtype="f16"),
        # the benchmark's step: a graph of 65 k nodes that fits the caches, repeated
        dict(name="step_rmat16", op="step", pattern="rmat", scale=16, edge_factor=16, d=32, N=128, dtype="f16"),
        # a regular mesh operator applied to a block of vectors
        dict(name="spmm_stencil_1024", op="spmm", pattern="stencil", grid=1024, N=64, dtype="f16"),
        # feature aggregation over a power-law graph of a million nodes
        dict(name="spmm_rmat20", op="spmm", pattern="rmat", scale=20, edge_factor=32, N=128, dtype="bf16"),
        # inference of an attention layer over a graph of 262 k nodes
        dict(name="attention_lognormal", op="attention", pattern="lognormal", M=262144, d=64, N=256, dtype="f16"),
        # a training step of that layer
        dict(name="train_lognormal", op="train", pattern="lognormal", M=262144, d=64, N=256, dtype="f16"),
        # link scores of a graph of 262 k nodes, long features
        dict(name="scores_rmat18", op="scores", pattern="rmat", scale=18, edge_factor=16, d=128, dtype="bf16"),
        # a rectangular (bipartite) matrix of odd sizes whose weights change, a width that is no power of two
        dict(name="reweight_odd", op="reweight", pattern="uniform", M=100003, K=50021, deg=11, N=200, dtype="bf16"),
        # preparing a graph: small, where launches and synchronisations count, and large
        dict(name="convert_rmat16", op="convert", pattern="rmat", scale=16, edge_factor=16, dtype="f16"),
        dict(name="convert_rmat20", op="convert", pattern="rmat", scale=20, edge_factor=32, dtype="bf16"),
        # what a backward pass prepares on top
        dict(name="transpose_lognormal", op="transpose", pattern="lognormal", M=262144, dtype="f16"),
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["spmm", "spmm", "step", "attention", "attention", "train", "scores", "reweight", "convert", "transpose"])
    pattern = rng.choice(["uniform", "rmat", "rmat", "stencil", "lognormal"])
    case = dict(op=op, pattern=pattern)
    if pattern == "uniform":
        case.update(M=spread(1500, 90000 if op == "train" else 200000), K=spread(1500, 200000), deg=rng.randint(3, 40))
    elif pattern == "rmat":
        scale = rng.randint(12, 17 if op == "train" else 19)
        case.update(scale=scale, edge_factor=rng.randint(6, 32 if scale < 19 else 20))
    elif pattern == "stencil":
        case.update(grid=spread(60, 500 if op == "train" else 900))
    else:
        case.update(M=spread(2000, 150000 if op == "train" else 250000))
    if op in ("spmm", "step", "attention", "train", "reweight"):
        case["N"] = 8 * spread(2, 32)  # 16 .. 256 columns, odd multiples of eight among them
    if op in ("step", "attention", "train"):
        case["d"] = 8 * spread(2, 16)  # 16 .. 128 features
    if op == "scores":
        case["d"] = 8 * spread(2, 32)
    case["dtype"] = rng.choice(["f16", "bf16"])
    return case


# --------------------------------------------------------------------------------------------------- inputs
def _shape(case):
    if case["pattern"] == "uniform":
        return case["M"], case["K"]
    n = {"rmat": lambda: 1 << case["scale"], "stencil": lambda: case["grid"] ** 2, "lognormal": lambda: case["M"]}[case["pattern"]]()
    return n, n


def _torch_dtype(case):
    return torch.float16 if case["dtype"] == "f16" else torch.bfloat16


def _csr(case, turn):
    """(rowptr, colidx): int32 on the GPU, columns ascending in each row, no duplicates.  The draws belong to the
    case, so that a case always has the same number of entries and vectors; its columns are numbered from
    another one on for each ``turn`` (a mesh has one numbering)."""
    M, K = _shape(case)
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(0)
    if case["pattern"] == "uniform":
        rows = torch.arange(M, device=dev).repeat_interleave(case["deg"])
        cols = torch.randint(0, K, (rows.numel(),), generator=gen, device=dev)
    elif case["pattern"] == "lognormal":
        deg = torch.exp(torch.randn(M, generator=gen, device=dev) + 2.5).round().clamp(1, min(4096, K)).to(torch.int64)
        rows = torch.arange(M, device=dev).repeat_interleave(deg)
        cols = torch.randint(0, K, (rows.numel(),), generator=gen, device=dev)
    elif case["pattern"] == "rmat":
        a, b, c, _ = RMAT
        n = case["edge_factor"] << case["scale"]
        rows = torch.zeros(n, dtype=torch.int64, device=dev)
        cols = torch.zeros(n, dtype=torch.int64, device=dev)
        for _ in range(case["scale"]):
            u = torch.rand(n, generator=gen, device=dev)
            rows = rows * 2 + (u >= a + b)
            cols = cols * 2 + (((u >= a) & (u < a + b)) | (u >= a + b + c))
    else:
        g = case["grid"]
        i = torch.arange(g * g, device=dev)
        x, y = i % g, i // g
        rows = torch.cat([i, i[x > 0], i[x < g - 1], i[y > 0], i[y < g - 1]])
        cols = torch.cat([i, i[x > 0] - 1, i[x < g - 1] + 1, i[y > 0] - g, i[y < g - 1] + g])
    if case["pattern"] != "stencil":
        cols = (cols + turn) % K
    key = torch.unique(rows * K + cols)  # sorted: CSR order
    rowptr = torch.searchsorted(key, torch.arange(M + 1, device=dev) * K).to(torch.int32)
    return rowptr, (key % K).to(torch.int32)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt, op = _torch_dtype(case), case["op"]
    M, K = _shape(case)
    rowptr, colidx = _csr(case, int(torch.randint(0, K, (1,), generator=gen, device="cuda")))
    nnz = colidx.numel()

    def normal(rows, cols, std=1.0):
        return (torch.randn((rows, cols), generator=gen, device="cuda") * std).to(dt)

    # edge weights of a graph lie in (0, 1), a mesh operator's coefficients have either sign
    vals = (torch.rand(nnz, generator=gen, device="cuda") if case["pattern"] in ("rmat", "lognormal")
            else torch.randn(nnz, generator=gen, device="cuda")).to(dt)
    s = dict(op=op, M=M, K=K, rowptr=rowptr, colidx=colidx, vals=vals)
    if op in ("convert", "transpose"):
        return s
    with_values = op == "spmm" or op == "step"
    s["fmt"] = fmt = fs.fs_convert(rowptr, colidx, vals if with_values else None, M, K, torch_dtype=dt)
    if op in ("spmm", "step", "reweight"):
        s["B"] = normal(K, case["N"])
    if op in ("step", "scores"):
        s["X"], s["Y"] = normal(M, case["d"]), normal(K, case["d"])
    if op == "step":
        work = torch.empty(max(fs.fs_spmm_workspace_bytes(fmt, case["N"]), 16), dtype=torch.uint8, device="cuda")
        s["scores"] = torch.empty(fmt.V * fmt.nvec, dtype=dt, device="cuda")
        s["C"] = torch.empty((M, case["N"]), dtype=dt, device="cuda")
        s["sddmm"] = fs.bind_sddmm(fmt, s["X"], s["Y"], out=s["scores"])
        s["spmm"] = fs.bind_spmm(fmt, s["B"], out=s["C"], work=work)
    if op in ("attention", "train"):
        s["X"], s["Y"] = normal(M, case["d"], 8 ** -0.5), normal(K, case["d"], 8 ** -0.5)
        s["H"] = normal(K, case["N"])
        s["scale"] = case["d"] ** -0.5
    if op == "train":
        s["dOut"] = normal(M, case["N"])
        rowptr_t, colidx_t, s["perm"] = fs.fs_csr_transpose(rowptr, colidx, M, K)
        s["fmt_t"] = fs.fs_convert(rowptr_t, colidx_t, None, K, M, torch_dtype=dt)
    return s


# ------------------------------------------------------------------------------------------------- one pass
def run(s):
    op = s["op"]
    if op == "convert":
        f = fs.fs_convert(s["rowptr"], s["colidx"], s["vals"], s["M"], s["K"])
        # the arrays of the format; the work list beside them is a schedule and changes no result
        return {"win_ptr": f.win_ptr_t(), "vec_col": f.vec_col_t(), "vec_mask": f.vec_mask_t(), "csr_to_slot": f.csr_to_slot_t(),
                "vals_blk": f.vals_blk_t(), "blk_desc": f.blk_desc_t(), "blk_row_base": f.blk_row_base_t()}
    if op == "transpose":
        rowptr_t, colidx_t, perm = fs.fs_csr_transpose(s["rowptr"], s["colidx"], s["M"], s["K"])
        return {"rowptr_t": rowptr_t, "colidx_t": colidx_t, "perm": perm, "vals_t": fs.fs_gather16(s["vals"], perm)}
    fmt = s["fmt"]
    if op == "spmm":
        return fs.fs_spmm(fmt, s["B"])
    if op == "step":
        return s["sddmm"](), s["spmm"]()
    if op == "attention":
        return fs.fs_attention(fmt, s["X"], s["Y"], s["H"], scale=s["scale"])
    if op == "scores":
        return fs.fs_sddmm(fmt, s["X"], s["Y"], blocked=False)
    if op == "reweight":
        return fs.fs_spmm(fmt, s["B"], vals=fs.fs_csr_to_blk(fmt, s["vals"]))
    # train: forward
    X, Y, H, dOut, scale, fmt_t = s["X"], s["Y"], s["H"], s["dOut"], s["scale"], s["fmt_t"]
    P = fs.fs_edge_softmax(fmt, fs.fs_sddmm(fmt, X, Y), scale=scale)
    out = fs.fs_spmm(fmt, H, vals=P)
    # backward: G arrives at P, dS at the scores; the gradients of Y and H are products on A^T's format
    G = fs.fs_sddmm(fmt, dOut, H)
    dS = fs.fs_edge_softmax_backward(fmt, P, G, scale=scale)
    dX = fs.fs_spmm(fmt, Y, vals=dS)

    def carried(blk):
        return fs.fs_csr_to_blk(fmt_t, fs.fs_gather16(fs.fs_blk_to_csr(fmt, blk), s["perm"]))

    dY = fs.fs_spmm(fmt_t, X, vals=carried(dS))
    dH = fs.fs_spmm(fmt_t, dOut, vals=carried(P))
    return {"out": out, "dX": dX, "dY": dY, "dH": dH}


# ------------------------------------------------------------------------- what a pass cannot do without
def _expected_cells(case, row_bits=0):
    """Expected number of distinct (row >> row_bits, column) cells that hold an entry: the stored entries for
    row_bits = 0, the nonzero vectors of windows of 2^row_bits rows otherwise, the referenced columns where
    row_bits covers all rows (row_bits None)."""
    M, K = _shape(case)

    def hit(p, n):  # probability that at least one of n draws falls into a cell of probability p
        return -math.expm1(n * math.log1p(-p)) if p < 1 else 1.0

    if case["pattern"] in ("uniform", "lognormal"):
        deg = case["deg"] if case["pattern"] == "uniform" else math.exp(3.0)
        rows = M if row_bits is None else min(M, 1 << row_bits)
        return M / rows * K * hit(1.0 / K, deg * rows)
    if case["pattern"] == "stencil":
        g = case["grid"]
        if row_bits is None:
            return K
        return 5 * g * g - 4 * g if row_bits == 0 else M / (1 << row_bits) * (3 * (1 << row_bits) + 2)
    a, b, _, d = RMAT  # b == c: cells differ only in how many levels took a, d, or either of the other two
    levels = case["scale"]
    free = levels if row_bits is None else row_bits  # levels whose row bit is summed over
    n, total = case["edge_factor"] << levels, 0.0
    for i in range(levels - free + 1):
        for j in range(levels - free - i + 1):
            k = levels - free - i - j
            cells = math.comb(levels - free, i) * math.comb(levels - free - i, j) * 2.0 ** k
            for m in range(free + 1):
                p = a ** i * d ** j * b ** k * (a + b) ** m * (b + d) ** (free - m)
                total += cells * math.comb(free, m) * hit(p, n)
    return total


def work(case):
    M, K = _shape(case)
    op, nnz = case["op"], _expected_cells(case)
    N, d = case.get("N", 0), case.get("d", 0)
    pattern = 4 * nnz + 4 * (M + 1)  # column indices and row pointers
    cols = min(K, _expected_cells(case, None))  # columns that are referenced: rows of B, Y and H that are read
    if op == "convert":
        nvec, V = _expected_cells(case, 3), 8
        if nnz >= 1 << 22 and nnz >= 12 * M and nvec * 20 > nnz * 19:  # large, and rows share no columns: four-row windows
            nvec, V = _expected_cells(case, 2), 4
        blocks = nvec / 32 + M / V / 2
        return {"bytes": pattern + 2 * nnz + 4 * M / V + 8 * nvec + 4 * nnz + 2 * V * nvec + blocks * (16 + 4 * V), "flops": 0}
    if op == "transpose":
        return {"bytes": pattern + 2 * nnz + 4 * (K + 1) + 10 * nnz, "flops": 0}
    if op in ("spmm", "reweight"):
        return {"bytes": pattern + 2 * nnz + 2 * N * (cols + M), "flops": 2 * nnz * N}
    if op == "scores":
        return {"bytes": pattern + 2 * d * (M + cols) + 2 * nnz, "flops": 2 * nnz * d}
    if op == "step":
        return {"bytes": pattern + 2 * d * (M + cols) + 2 * nnz + 2 * nnz + 2 * N * (cols + M), "flops": 2 * nnz * (d + N)}
    if op == "attention":
        return {"bytes": pattern + 2 * d * (M + cols) + 2 * N * (cols + M), "flops": 2 * nnz * (d + N)}
    # train: X, Y, H and dOut read, out and three gradients written; A and A^T with the map between them
    return {"bytes": 3 * pattern + 2 * d * 2 * (M + cols) + 2 * N * 2 * (M + cols), "flops": 6 * nnz * (d + N)}


def tolerance(case):
    if case["op"] in ("convert", "transpose"):
        return "exact"
    # one rounding to the element type of an fp32 sum, whose order is free: half an ulp of either side.  In
    # attention and training the probabilities are rounded on the way, in training the scores and the gradients as
    # well (twice as many roundings).
    stages = {"attention": 2, "train": 4}.get(case["op"], 1)
    return {"rel": stages * (5e-4 if case["dtype"] == "f16" else 4e-3)}
