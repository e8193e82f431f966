"""SDDMM at the feature counts where its kernel changes or ends a chunk raggedly, bit for bit on exact inputs
(every product and partial sum is a multiple of 1/2 far below 2^24), and in both orders in which blocks are taken."""
import numpy as np
import pytest

import oracle
from gpu_util import from_dev_bits, to_dev, upload_csr
from test_gpu_exact import fs, halves, hub_matrix, int_dense, same_bits  # noqa: F401
from workloads import Dense, csr_from_coo, stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [8, 32, 40, 64, 72, 128, 136, 248, 256, 264, 392])
@pytest.mark.parametrize("V", [4, 8, 16])
def test_sddmm_widths_bit_exact(fs, d, V):  # noqa: F811
    import torch
    dtype = "f16" if (d // 8 + V // 4) % 2 else "bf16"
    lim = 1 if dtype == "bf16" else 2  # scores are multiples of 1/2; bf16 rounds those above 64, like the oracle
    A = hub_matrix(77, 6500, dtype, seed=V + d)
    X = Dense(halves(stream(V + d, 97, 2), (A.M, d), -lim, lim, dtype), dtype)
    Y = int_dense(A.K, d, dtype, seed=V + d, tid=3, lim=lim)
    ref, _ = oracle.sddmm(A.M, A.K, A.rowptr, A.colidx, X.bits, Y.bits, dtype, want_scale=False)
    want = oracle.round_f64_to_bits(ref, dtype)
    rp, ci, _ = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, None, A.M, A.K, torch_dtype=torch.float16 if dtype == "f16" else torch.bfloat16, V=V, chunk=64)
    assert fmt.n_cut_items * 8 >= fmt.n_items
    Xd, Yd = to_dev(X.bits, dtype), to_dev(Y.bits, dtype)
    wide = torch.zeros((A.K, d + 1024), dtype=Yd.dtype, device="cuda")  # beyond 4 MB
    wide[:, :d] = Yd
    for Yv in (Yd, wide[:, :d]):
        blk = fs.fs_sddmm(fmt, Xd, Yv)
        same_bits(from_dev_bits(fs.fs_blk_to_csr(fmt, blk)), want, "fs_sddmm V=%d d=%d" % (V, d))
        got = from_dev_bits(blk).copy()
        got[fmt.csr_to_slot_t().cpu().numpy()] = 0
        assert not got.any(), "positions outside the pattern must be +0.0"
        same_bits(from_dev_bits(fs.fs_sddmm(fmt, Xd, Yv, blocked=False)), want, "fs_sddmm, CSR order, V=%d d=%d" % (V, d))


@pytest.mark.parametrize("d", [32, 40, 64, 128, 264])
@pytest.mark.parametrize("V,dtype", [(8, "f16"), (16, "bf16")])
@pytest.mark.parametrize("kind", ["hubs", "some hubs", "few items"])
def test_sddmm_block_order(fs, kind, V, dtype, d):  # noqa: F811
    """Enough items and enough of Y for launch order (all items parts of hub windows; one in five, which d <= 32 leaves
    in slot order), and the same hubs with too few items for it."""
    import torch
    K = 70000  # more than 4 MB of Y from d = 32 on
    hubs, n, short = {"hubs": (2 * V, 60000, 0), "some hubs": (V, 60000, 60000), "few items": (V, 3000, 3)}[kind]
    rng = stream(V + d, 95, 1)
    cols = [rng.choice(K, size=n, replace=False) for _ in range(hubs)]
    rows = [np.full(n, i) for i in range(hubs)]
    rows.append(hubs + np.arange(short))
    cols.append(rng.integers(0, K, size=short))
    A = csr_from_coo(hubs + short, K, np.concatenate(rows), np.concatenate(cols), "u11", dtype, rng)
    lim = 1 if dtype == "bf16" else 2
    X = Dense(halves(stream(V + d, 95, 2), (A.M, d), -lim, lim, dtype), dtype)
    Y = int_dense(K, d, dtype, seed=V + d, tid=4, lim=lim)
    ref, _ = oracle.sddmm(A.M, A.K, A.rowptr, A.colidx, X.bits, Y.bits, dtype, want_scale=False)
    want = oracle.round_f64_to_bits(ref, dtype)
    rp, ci, _ = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, None, A.M, A.K, torch_dtype=torch.float16 if dtype == "f16" else torch.bfloat16, V=V, chunk=32)
    cut, items = fmt.n_cut_items, fmt.n_items
    assert {"hubs": items >= 4096 and cut * 4 >= items * 3, "some hubs": items >= 4096 and items <= 8 * cut and cut * 2 < items,
            "few items": items < 1536}[kind], (cut, items)
    Xd, Yd = to_dev(X.bits, dtype), to_dev(Y.bits, dtype)
    same_bits(from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_sddmm(fmt, Xd, Yd))), want, "fs_sddmm")
    same_bits(from_dev_bits(fs.fs_sddmm(fmt, Xd, Yd, blocked=False)), want, "fs_sddmm, CSR order")


@pytest.mark.parametrize("d", [136, 160, 168, 232, 256])
@pytest.mark.parametrize("V", [4, 8, 16])
@pytest.mark.parametrize("ordered", [False, True])
def test_sddmm_whole_rows(fs, ordered, V, d):  # noqa: F811
    """Eight to ten thousand blocks, from which on windows of sixteen rows gather rows of up to 512 bytes whole and lower ones still
    take chunks (test_sddmm_whole_rows_by_height has more): short windows, hubs of many blocks whose rows of X stay,
    empty windows between them, a last window of fewer than V rows; in slot order and in launch order."""
    import torch
    dtype = "bf16" if (d // 8 + V // 4) % 2 else "f16"
    rng = stream(V + d, 94, 1)
    K, hubs, n, short = (60000, 5 * V, 60000, 0) if ordered else (30000, V, 700, 8300 * V)  # ordered: 9375 blocks
    rows = [np.full(n, i) for i in range(hubs)] + [hubs + 3 * V + np.arange(short)]
    cols = [rng.choice(K, size=n, replace=False) if not ordered else np.arange(n) for _ in range(hubs)] + [rng.integers(0, K, size=short)]
    if not ordered:
        rows.append(hubs + 3 * V + np.arange(short))
        cols.append(rng.integers(0, K, size=short))
    A = csr_from_coo(hubs + 3 * V + short + 3, K, np.concatenate(rows), np.concatenate(cols), "u11", dtype, rng)
    lim = 1 if dtype == "bf16" else 2
    X = Dense(halves(stream(V + d, 94, 2), (A.M, d), -lim, lim, dtype), dtype)
    Y = int_dense(K, d, dtype, seed=V + d, tid=5, lim=lim)
    ref, _ = oracle.sddmm(A.M, A.K, A.rowptr, A.colidx, X.bits, Y.bits, dtype, want_scale=False)
    want = oracle.round_f64_to_bits(ref, dtype)
    rp, ci, _ = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, None, A.M, A.K, torch_dtype=torch.float16 if dtype == "f16" else torch.bfloat16, V=V, chunk=64)
    assert fmt.n_blocks >= 8192 and (fmt.n_items >= 4096 and fmt.n_cut_items * 8 >= fmt.n_items) == ordered, (fmt.n_blocks, fmt.n_items, fmt.n_cut_items)
    Xd, Yd = to_dev(X.bits, dtype), to_dev(Y.bits, dtype)
    same_bits(from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_sddmm(fmt, Xd, Yd))), want, "fs_sddmm")
    same_bits(from_dev_bits(fs.fs_sddmm(fmt, Xd, Yd, blocked=False)), want, "fs_sddmm, CSR order")


@pytest.mark.parametrize("d", [136, 168, 200, 248])
@pytest.mark.parametrize("V,kind", [(4, "short"), (8, "short"), (16, "short"), (4, "hubs"), (8, "hubs"), (16, "hubs")])
def test_sddmm_whole_rows_by_height(fs, V, kind, d):  # noqa: F811
    """Block counts from which rows are gathered whole at each window height: windows of three blocks (the last one narrow) in slot
    order, and hub windows, one long row each, in launch order.  Exact in fp32, so bit for bit."""
    import torch
    dtype = "bf16" if (d // 8 + V // 4) % 2 else "f16"
    rng = np.random.default_rng(V + d)
    K = 30000
    if kind == "short":
        W = {4: 11000, 8: 4400, 16: 2800}[V]
        rows = np.repeat(np.arange(W * V), 88 // V)
        cols = rng.integers(0, K, size=rows.shape[0])
    else:
        W = {4: 120, 8: 24, 16: 16}[V]
        rows, cols = np.repeat(np.arange(W) * V + 1, 18000), np.concatenate([rng.choice(K, size=18000, replace=False) for _ in range(W)])
    A = csr_from_coo(W * V, K, rows, cols, "u11", dtype, rng)
    lim = 1 if dtype == "bf16" else 2
    X = Dense(halves(stream(V + d, 95, 2), (A.M, d), -lim, lim, dtype), dtype)
    Y = int_dense(K, d, dtype, seed=V + d, tid=6, lim=lim)
    ref, _ = oracle.sddmm(A.M, A.K, A.rowptr, A.colidx, X.bits, Y.bits, dtype, want_scale=False)
    want = oracle.round_f64_to_bits(ref, dtype)
    rp, ci, _ = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, None, A.M, A.K, torch_dtype=torch.float16 if dtype == "f16" else torch.bfloat16, V=V, chunk=64 if V > 4 else 256)
    assert fmt.n_blocks >= {4: 1 << 15 if kind == "short" else 1 << 16, 8: 12800, 16: 8192}[V] and fmt.nvec >= 18 * fmt.n_blocks, (fmt.n_blocks, fmt.nvec)
    Xd, Yd = to_dev(X.bits, dtype), to_dev(Y.bits, dtype)
    same_bits(from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_sddmm(fmt, Xd, Yd))), want, "fs_sddmm")
    same_bits(from_dev_bits(fs.fs_sddmm(fmt, Xd, Yd, blocked=False)), want, "fs_sddmm, CSR order")
