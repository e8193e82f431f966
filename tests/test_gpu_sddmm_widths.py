"""SDDMM at the feature counts where its kernel changes or ends a chunk raggedly, bit for bit on exact inputs
(every product and partial sum is a multiple of 1/2 far below 2^24), in both orders in which blocks are taken: Y
within one XCD's L2, and rows so far apart that it is not (hub windows then go in launch order)."""
import numpy as np
import pytest

import oracle
from gpu_util import from_dev_bits, to_dev, upload_csr
from test_gpu_exact import fs, halves, hub_matrix, int_dense, same_bits  # noqa: F401
from workloads import Dense, stream

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
