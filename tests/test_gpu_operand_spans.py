"""Dense operands whose rows lie far apart, where the byte offset of a row changes its kind: from 2 GiB on it no longer fits
a signed 32-bit number, from 4 GiB on no 32-bit number at all (the kernels then take 64-bit addresses), and a pitch of 4 GiB
does not fit one either.  Exact inputs (every product and partial sum is a multiple of 1/2 far below 2^24), bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import from_dev_bits, to_dev, upload_csr
from test_gpu_exact import fs, halves, int_dense, same_bits  # noqa: F401
from workloads import Dense, random_csr, stream

pytestmark = pytest.mark.gpu
FAR = 70000  # rows of the operand that spans far


def far_rows(t, pitch):
    """``t`` with its rows ``pitch`` elements apart."""
    import torch
    base = torch.zeros((t.shape[0], pitch), dtype=t.dtype, device="cuda")
    base[:, :t.shape[1]] = t
    return base[:, :t.shape[1]]


@pytest.mark.parametrize("d", [32, 64, 128, 264])
@pytest.mark.parametrize("which", ["X", "Y"])
@pytest.mark.parametrize("pitch", [16384, 32768])  # elements: 2.3 GB and 4.6 GB
def test_sddmm_far_rows(fs, pitch, which, d):  # noqa: F811
    import torch
    M, K = (FAR, 300) if which == "X" else (300, FAR)
    A = random_csr(M, K, 0.002, "f16", seed=78)
    far = np.repeat(np.arange(M), np.diff(A.rowptr)) if which == "X" else A.colidx
    assert int(far.max()) * pitch * 2 >= 2 ** 31  # rows near the far end are read
    X = Dense(halves(stream(d, 90, 1), (M, d), -2, 2, "f16"), "f16")
    Y = int_dense(K, d, "f16", seed=d, tid=2, lim=2)
    ref, _ = oracle.sddmm(M, K, A.rowptr, A.colidx, X.bits, Y.bits, "f16", want_scale=False)
    want = oracle.round_f64_to_bits(ref, "f16")
    rp, ci, _ = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, None, M, K, torch_dtype=torch.float16)
    Xd, Yd = to_dev(X.bits, "f16"), to_dev(Y.bits, "f16")
    if which == "X":
        Xd = far_rows(Xd, pitch)
    else:
        Yd = far_rows(Yd, pitch)
    same_bits(from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_sddmm(fmt, Xd, Yd))), want, "fs_sddmm")
    same_bits(from_dev_bits(fs.fs_sddmm(fmt, Xd, Yd, blocked=False)), want, "fs_sddmm, CSR order")
    del Xd, Yd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d", [32, 64, 128, 264])
@pytest.mark.parametrize("which", ["X", "Y"])
def test_sddmm_rows_of_4_gib(fs, which, d):  # noqa: F811
    import torch
    M, K = (3, 40) if which == "X" else (40, 3)
    A = random_csr(M, K, 0.5, "f16", seed=80)
    rp, ci, _ = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, None, M, K, torch_dtype=torch.float16)
    X, Y = (torch.randint(-2, 3, (n, d), device="cuda").half() for n in (M, K))
    want = fs.fs_sddmm(fmt, X, Y)
    pitch = (1 << 31) + 8
    base = torch.empty(2 * pitch + d, dtype=torch.float16, device="cuda")
    far = torch.as_strided(base, (3, d), (pitch, 1))
    far.copy_(X if which == "X" else Y)
    base[d:2 * d] = float("nan")  # where a pitch cut to 32 bits would look
    got = fs.fs_sddmm(fmt, far, Y) if which == "X" else fs.fs_sddmm(fmt, X, far)
    same_bits(from_dev_bits(got), from_dev_bits(want), "fs_sddmm")
    del base, far
    torch.cuda.empty_cache()


def test_products_far_rows(fs):  # noqa: F811
    """SpMM and the fused attention kernel on the same spans: the bits of the close-lying operand."""
    import torch
    A = random_csr(300, FAR, 0.002, "f16", seed=79)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, A.M, A.K)
    gen = torch.Generator(device="cuda").manual_seed(3)
    X, Y, H = (torch.randn((r, n), generator=gen, device="cuda").half() for r, n in ((A.M, 64), (FAR, 64), (FAR, 128)))
    far = far_rows(H, 16384)
    same_bits(from_dev_bits(fs.fs_spmm(fmt, far)), from_dev_bits(fs.fs_spmm(fmt, H)), "fs_spmm")
    want = from_dev_bits(fs.fs_attention(fmt, X, Y, H, 0.125))
    same_bits(from_dev_bits(fs.fs_attention(fmt, X, Y, far, 0.125)), want, "fs_attention, H")
    same_bits(from_dev_bits(fs.fs_attention(fmt, X, far_rows(Y, 16384), H, 0.125)), want, "fs_attention, Y")
    del far
    torch.cuda.empty_cache()
