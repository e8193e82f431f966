"""The conversion where its units of work change: windows just below and above what one wavefront takes, hub windows cut
by columns (rows alike, one long row, identical rows, a longest row that says nothing about the others), groups of tiny
and empty windows, a single row per window, every array bit for bit against the reference converter."""
import numpy as np
import pytest

import oracle
from gpu_util import upload_csr
from test_gpu_parity import assert_format_equal, assert_items_valid, assert_row_base_valid, fs  # noqa: F401
from workloads import Csr, csr_from_coo, stream

pytestmark = pytest.mark.gpu


def from_rows(rows, K, dtype="f16"):
    """CSR with the given columns per row."""
    r = np.repeat(np.arange(len(rows)), [len(c) for c in rows])
    c = np.concatenate(rows) if len(r) else np.zeros(0, dtype=np.int64)
    return csr_from_coo(len(rows), K, r, c, "u11", dtype, stream(3, 94, len(rows)))


def pattern(kind, V, rng):
    K = 40000
    pick = lambda n, lo=0, hi=K: np.sort(rng.choice(hi - lo, size=n, replace=False)) + lo  # noqa: E731
    rows = []
    if kind == "edges":  # windows of 511, 512, 513 and 514 entries, then one entry, then none
        for total in (511, 512, 513, 514, 1):
            for r in range(V):
                rows.append(pick((total + V - 1 - r) // V))
        rows += [pick(0)] * V
    elif kind == "alike":
        rows = [pick(900) for _ in range(2 * V)]
    elif kind == "one long row":
        rows = [pick(20000)] + [pick(3) for _ in range(V - 1)] + [pick(7) for _ in range(V)]
    elif kind == "identical":  # every vector full
        c = pick(1500)
        rows = [c] * V + [pick(2)] * V
    elif kind == "apart":  # the longest row's columns lie before all others'
        rows = [np.arange(3000)] + [pick(2500, 10000) for _ in range(V - 1)]
    elif kind == "dense start":  # all rows hold the first columns, then thin out
        rows = [np.unique(np.concatenate([np.arange(700), pick(300 * (r % 3 + 1))])) for r in range(2 * V)]
    elif kind == "runs":  # runs of 1, 2, 4 ... windows, hubs between them, a last group cut short (what just fits a unit depends on
        # the matrix' entries: test_convert_units_of_so_many_entries)
        group = 64 // (1 << (V - 1).bit_length()) if V > 1 else 16
        sizes = [0] * group + [512 // group] * group + [512 // group + 1] * group      # a whole group fits, exactly and not
        sizes += [256, 256] * (group // 2) + [257, 256] * (group // 2)                 # pairs
        sizes += ([1, 511, 512, 0, 600, 3, 509, 700, 2, 513, 1, 1, 400, 112, 113, 2000] * 2)[:max(group, 3)]
        sizes += [5] * (group // 2 + 1)
        for n in sizes:
            rows += [pick((n + V - 1 - r) // V) for r in range(V)]
    elif kind == "few":  # units of 0 to 70 entries: up to 64 an entry has a lane of its own; many share a column
        group = 1
        while group < 16 and (2 * group) * V <= 64:
            group *= 2
        for n in (0, 1, 2, 3, 31, 62, 63, 64, 65, 66, 70, 64, 5):
            at = np.sort(rng.integers(0, group * V, n))
            rows += [pick(int((at == r).sum()), 0, 90 if n % 2 else K) for r in range(group * V)]
    else:  # tiny: windows of a handful of entries and empty ones, ragged end
        rows = [pick(int(rng.integers(0, 3))) if rng.random() < 0.6 else pick(0) for _ in range(37 * V + max(V - 3, 0))]
    return from_rows(rows, K)


@pytest.mark.parametrize("V,KB", [(1, 32), (2, 32), (4, 32), (8, 32), (16, 32), (32, 32), (3, 8), (8, 5)])
@pytest.mark.parametrize("kind", ["edges", "alike", "one long row", "identical", "apart", "dense start", "runs", "few", "tiny"])
def test_convert_units_bit_exact(fs, kind, V, KB):  # noqa: F811
    A = pattern(kind, V, np.random.default_rng(V * 100 + KB))
    rp, ci, va = upload_csr(A)
    for vals in (va, None):
        fmt = fs.fs_convert(rp, ci, vals, A.M, A.K, torch_dtype=va.dtype, V=V, KB=KB)
        ref = assert_format_equal(fmt, A, V, KB, with_vals=vals is not None)
        assert_items_valid(fmt)
        assert_row_base_valid(fmt, A)
        if KB == 32:  # the occupancy masks, seen from the rows
            desc = fmt.blk_desc_t().cpu().numpy().astype(np.int64)
            want = np.zeros((fmt.n_blocks, V), dtype=np.uint32)
            for x, (s, kf, _, _) in enumerate(desc):
                m = ref.vec_mask[s:s + (kf & 255)]
                for r in range(V):
                    want[x, r] = int(((m >> np.uint32(r)) & np.uint32(1)) @ (np.uint32(1) << np.arange(len(m), dtype=np.uint32))) if len(m) else 0
            assert np.array_equal(fmt.blk_row_bits_t().cpu().numpy().view(np.uint32), want)


@pytest.mark.parametrize("V,fill", [(1, 128), (2, 512), (4, 128), (4, 512), (8, 128), (8, 300), (8, 512), (16, 128), (16, 512), (32, 512)])
def test_convert_units_of_so_many_entries(fs, V, fill):  # noqa: F811
    """How full a unit of several windows gets depends on the matrix' entries: runs of windows that just fit and just do not, with
    as many entries around them as make that limit 128, 300 or 512."""
    rng = np.random.default_rng(V + fill)
    K = 40000
    pick = lambda n: np.sort(rng.choice(K, size=n, replace=False))  # noqa: E731
    group = min(64 // (1 << (V - 1).bit_length()) if V > 1 else 16, 16)
    sizes = [fill // group] * group + [fill // group + 1] * group + [fill // 2] * 4 + [fill // 2, fill // 2 + 1] * 4 + [fill, fill + 1, 0, 513, 3] * group
    rows = []
    for n in sizes:
        rows += [pick((n + V - 1 - r) // V) for r in range(V)]
    around = max(fill * 1024 + 600 - sum(len(r) for r in rows), 0) if fill > 128 else 0
    rows += [pick(20000) for _ in range(around // 20000)] + [pick(around % 20000), pick(5)]
    A = from_rows(rows, K)
    assert min(max(A.nnz // 1024, 128), 512) == fill
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, A.M, A.K, V=V)
    assert_format_equal(fmt, A, V, 32)
    assert_items_valid(fmt)
    assert_row_base_valid(fmt, A)


def test_convert_columns_beyond_26_bits_and_bad_hub_rows(fs):  # noqa: F811
    """Columns up to 2^31 - 2, and hub windows whose columns do not ascend: refused wherever the fault lies."""
    rng = np.random.default_rng(5)
    K = 2 ** 31 - 1
    rows = [np.sort(rng.choice(2 ** 31 - 2, size=n, replace=False)) for n in (900, 3, 400, 0, 70, 1, 2, 600, 5)]
    A = from_rows(rows, K)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, A.M, A.K, V=8)
    assert_format_equal(fmt, A, 8, 32)
    for row, at in ((0, 1), (0, 450), (0, 899), (2, 200), (7, 599), (8, 4)):
        bad = ci.clone()
        p = int(A.rowptr[row]) + at
        bad[p] = bad[p - 1]
        with pytest.raises(fs.FsError) as e:
            fs.fs_convert(rp, bad, va, A.M, A.K, V=8)
        assert e.value.code == 2
        bad = ci.clone()
        bad[int(A.rowptr[row]) + at] = -5
        with pytest.raises(fs.FsError) as e:
            fs.fs_convert(rp, bad, va, A.M, A.K, V=8)
        assert e.value.code == 2
    for i, v in ((3, 10 ** 9), (5, -1), (A.M, A.nnz - 1), (0, 1)):
        bad_rp = rp.clone()
        bad_rp[i] = v
        with pytest.raises(fs.FsError) as e:
            fs.fs_convert(bad_rp, ci, va, A.M, A.K, V=8)
        assert e.value.code == 2


@pytest.mark.parametrize("V", [0, 1, 4, 16])
def test_convert_no_rows_in_a_used_scratch_buffer(fs, V):  # noqa: F811
    """M = 0: the one window pointer is 0 whatever the scratch buffer held before."""
    import torch
    rp, none = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.empty(0, dtype=torch.int32, device="cuda")
    _, need = fs.fs_format_bytes(0, 0, V)
    scratch = torch.full((need,), 0x7F, dtype=torch.uint8, device="cuda")
    fmt = fs.fs_convert(rp, none, None, 0, 9, torch_dtype=torch.float16, V=V, scratch=scratch)
    assert fmt.win_ptr_t().tolist() == [0] and fmt.nvec == 0 and fmt.n_blocks == 0 and fmt.c.n_items == 0


def test_convert_more_units_than_one_launch_takes(fs):  # noqa: F811
    """2^28 mostly empty rows in windows of one: more than 2^24 units.  A window is a row, so win_ptr is the row pointer,
    every entry a vector of its own, in CSR order."""
    import torch
    M, K = (1 << 28) + 1000, 50000
    gen = torch.Generator(device="cuda").manual_seed(4)
    rows = torch.randint(0, M, (3000,), generator=gen, device="cuda")
    rows = torch.cat([rows, torch.tensor([0, 5, M - 1], device="cuda"), torch.full((1500,), M // 2, device="cuda")])  # one row is cut by columns
    key = torch.unique(rows * K + torch.randint(0, K, rows.shape, generator=gen, device="cuda"))
    ci = (key % K).to(torch.int32)
    counts = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    counts.index_add_(0, key // K + 1, torch.ones_like(ci))
    rp = torch.cumsum(counts, 0, dtype=torch.int32)
    del counts
    fmt = fs.fs_convert(rp, ci, torch.ones_like(ci, dtype=torch.float16), M, K, V=1)
    assert fmt.nvec == ci.numel() and torch.equal(fmt.win_ptr_t(), rp) and torch.equal(fmt.vec_col_t(), ci)
    assert torch.equal(fmt.csr_to_slot_t(), torch.arange(ci.numel(), dtype=torch.int32, device="cuda"))
    assert (fmt.vec_mask_t() == 1).all() and (fmt.vals_blk_t() == 1).all()
    del fmt, rp
    torch.cuda.empty_cache()


def work_list(wp, KB, T, chunk):
    """Item starts by their definition: every candidate (a multiple of Ts among the block slots) starts the part it lies in of
    a window that is cut, or an item at the nearer end of one that is not."""
    blk = np.concatenate([[0], np.cumsum(np.maximum(1, -(-np.diff(wp) // KB)))])
    NB, longest = blk[-1], np.diff(blk).max()
    Ts, starts = min(T, 4), []
    if chunk == 0:
        Ts = 2 if NB < 4096 else 3 if NB < 16384 else 4
        assert T == (4 if longest > 12 and NB < 5120 else 6 if longest > 12 and NB < 8192 else min(max(-(-NB // 4096), 8), 16))
    for x in range(0, blk[-1], Ts):
        w = np.searchsorted(blk, x, side="right") - 1
        lo, hi = blk[w], blk[w + 1]
        if hi - lo > T + T // 2:
            plen = -(-(hi - lo) // ((hi - lo + T // 2) // T))
            starts.append(lo + (x - lo) // plen * plen)
        else:
            starts.append(lo if x - lo <= hi - x else hi)
    return blk, np.unique(starts)


@pytest.mark.parametrize("chunk", [0, 32, 64, 96, 128, 160, 224, 1024])
@pytest.mark.parametrize("W", [1, 2, 1023, 1024, 1025, 2500, 5000])  # a workgroup takes 1024 windows; all grains of chunk 0
def test_convert_work_list_is_what_the_candidates_make(fs, W, chunk):  # noqa: F811
    V, K = 4, 30000
    rng = np.random.default_rng(W + chunk)
    sizes = rng.choice([0, 1, 20, 33, 90, 150, 260, 500, 2200, 9000], p=[.2, .3, .1, .1, .1, .08, .06, .04, .015, .005], size=W)
    sizes[rng.integers(0, W, 2)] = (7000, 400)
    rows = []
    for n in sizes:
        rows += [np.sort(rng.choice(K, size=(n + V - 1 - r) // V, replace=False)) for r in range(V)]
    A = from_rows(rows, K)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, A.M, A.K, V=V, KB=32, chunk=chunk)
    assert_format_equal(fmt, A, V, 32)
    assert_items_valid(fmt)
    wp = fmt.win_ptr_t().cpu().numpy().astype(np.int64)
    blk, starts = work_list(wp, 32, fmt.chunk // 32, chunk)
    ends = np.append(starts[1:], blk[-1])
    items, order = fmt.items_t().cpu().numpy().astype(np.int64), fmt.item_order_t().cpu().numpy()
    real = starts < blk[-1]
    assert len(items) == len(starts) and np.array_equal(items[real, 0], starts[real]) and np.array_equal(items[real, 1], (ends - starts)[real])
    assert (items[~real] == 0).all()
    # launch order: parts of cut windows by column, whole windows costliest first, stably
    w_at = np.searchsorted(blk, items[:, 0], side="right") - 1
    w_end = np.searchsorted(blk, items[:, 0] + items[:, 1] - 1, side="right") - 1
    cut = real & ((items[:, 0] > blk[w_at]) | (items[:, 0] + items[:, 1] < blk[w_end + 1]))
    cost = items[:, 1] + w_end - w_at + 1
    col = fmt.vec_col_t().cpu().numpy().astype(np.int64)[np.minimum(items[:, 3], fmt.nvec - 1)]
    key = np.where(~real, 0xFFFFFF, np.where(cut, (col << 16) // K, (129 - np.minimum(cost, 128)) << 16))
    assert np.array_equal(order, np.argsort(key, kind="stable")) and fmt.n_cut_items == cut.sum()
    assert np.array_equal(fmt.items_by_cost_t().cpu().numpy(), items[order])


@pytest.mark.parametrize("V", [1, 4, 8, 32])  # units of sixteen, sixteen, eight and two windows
@pytest.mark.parametrize("span", [1, 2, 31, 33, 1 << 9, (1 << 10) + 1, 1 << 14, (1 << 14) + 1, 1 << 19, (1 << 19) + 3, 1 << 24, (1 << 29) + 1, (1 << 31) - 2])
def test_convert_columns_that_span_so_much(fs, V, span):  # noqa: F811
    """Ranks where a level is added: the columns of a unit lie within `span`, both ends among them; short windows, a full unit, a hub."""
    K = 2 ** 31 - 1
    rng = np.random.default_rng(V + span % 1000)
    base = int(rng.integers(0, K - span)) if K > span else 0
    rows = []
    for n in [3] * 16 + [500] + [2000] + [0, 7, 1]:
        for r in range(V):
            c = np.unique(rng.integers(0, span, (n + V - 1 - r) // V))
            if r == V - 1 and n:
                c = np.unique(np.concatenate([c, [0, span - 1]]))
            rows.append(base + c)
    A = from_rows(rows, K)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, A.M, A.K, V=V)
    assert_format_equal(fmt, A, V, 32)
    assert_row_base_valid(fmt, A)


@pytest.mark.parametrize("width,height,dense_row,blocks_an_item", [(64, 64, False, 2), (128, 128, False, 2), (256, 256, False, 4), (256, 130, False, 4),
                                                                   (512, 300, False, 4), (256, 256, True, 2), (400, 400, True, 4)])
def test_whole_items_of_a_mesh_have_a_power_of_two_blocks(fs, width, height, dense_row, blocks_an_item):
    """Windows of one block: items of three would take 24 rows, and the rows that share operands, a width of the mesh apart, would meet in
    no L2 where the width is a power of two."""
    import torch
    n = width * height
    i = np.arange(n)
    x, y = i % width, i // width
    rows = np.concatenate([i, i[x > 0], i[x < width - 1], i[y > 0], i[y < height - 1]])
    cols = np.concatenate([i, i[x > 0] - 1, i[x < width - 1] + 1, i[y > 0] - width, i[y < height - 1] + width])
    if dense_row:  # one window of more than 12 blocks, which is cut
        rows, cols = np.concatenate([rows, np.full(n // 64, 77)]), np.concatenate([cols, np.arange(n // 64) * 64])
    key = np.unique(rows * n + cols)
    rp = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))])
    fmt = fs.fs_convert(torch.from_numpy(rp).int().cuda(), torch.from_numpy(key % n).int().cuda(), None, n, n, torch_dtype=torch.float16, V=8)
    items = fmt.items_t().cpu().numpy()
    cut = fmt.n_cut_items
    assert (cut > 0) == dense_row
    whole = items[np.sort(fmt.item_order_t().cpu().numpy()[cut:])]
    # the one next to a cut window and the last may be shorter or longer
    assert (whole[:, 1] == blocks_an_item).sum() >= len(whole) - 3, np.bincount(whole[:, 1])
