"""Calls that allocate their own result run through the native module: same bits as the calls that are given it, same
errors for what they do not take."""
import pytest
import torch

from gpu_util import upload_csr
from test_gpu_parity import fs  # noqa: F401
from workloads import random_csr

pytestmark = pytest.mark.gpu


def same(a, b):
    torch.cuda.synchronize()  # (the calls may have run on another stream than the comparison's)
    assert a.shape == b.shape and a.dtype == b.dtype and torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("M,K,density,chunk,dtype", [(40, 56, 0.2, 0, "f16"), (64, 900, 0.5, 64, "bf16"), (8, 8, 0.05, 0, "f16")])
def test_native_calls_match_calls_with_given_outputs(fs, M, K, density, chunk, dtype):  # noqa: F811
    A = random_csr(M, K, density, dtype, seed=7)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, M, K, chunk=chunk)
    dt = va.dtype
    assert chunk == 0 or fmt.n_split_items > 0  # a workspace is needed
    gen = torch.Generator(device="cuda").manual_seed(1)
    X, Y, B = (torch.randn((r, c), generator=gen, device="cuda").to(dt) for r, c in ((M, 40), (K, 40), (K, 48)))
    new = lambda *shape: torch.empty(shape, dtype=dt, device="cuda")  # noqa: E731
    side = torch.cuda.Stream()
    for stream in (None, side):
        same(fs.fs_spmm(fmt, B, stream=stream), fs.fs_spmm(fmt, B, out=new(M, 48), stream=stream))
        same(fs.fs_spmm(fmt, B[:, 8:24], stream=stream), fs.fs_spmm(fmt, B[:, 8:24], out=new(M, 16), stream=stream))
        torch.cuda.synchronize()
        S = fs.fs_sddmm(fmt, X, Y, stream=stream)
        same(S, fs.fs_sddmm(fmt, X, Y, out=new(fmt.V * fmt.nvec), stream=stream))
        csr = fs.fs_sddmm(fmt, X, Y, blocked=False, stream=stream)
        same(csr, fs.fs_sddmm(fmt, X, Y, blocked=False, out_csr=new(fmt.nnz), stream=stream))
        same(fs.fs_blk_to_csr(fmt, S, stream=stream), csr)
        same(fs.fs_csr_to_blk(fmt, csr, stream=stream), S)
        P = fs.fs_edge_softmax(fmt, S, scale=0.5, stream=stream)
        same(P, fs.fs_edge_softmax(fmt, S, out=torch.empty_like(S), scale=0.5, stream=stream))
        same(fs.fs_edge_softmax_backward(fmt, P, S, scale=0.5, stream=stream),
             fs.fs_edge_softmax_backward(fmt, P, S, out=torch.empty_like(S), scale=0.5, stream=stream))
        same(fs.fs_spmm(fmt, B, vals=P, stream=stream), fs.fs_spmm(fmt, B, vals=P, out=new(M, 48), stream=stream))
        for call in (fs.fs_attention, fs.fs_sddmm_spmm):
            same(call(fmt, X, Y, B, 0.25, stream=stream), call(fmt, X, Y, B, 0.25, out=new(M, 48), stream=stream))
        idx = torch.arange(fmt.nnz - 1, -1, -1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()  # idx was made on the current stream
        same(fs.fs_gather16(va, idx, stream=stream), va.flip(0))


def test_native_calls_refuse_what_the_others_refuse(fs):  # noqa: F811
    A = random_csr(40, 56, 0.2, "f16", seed=7)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, 40, 56)
    t = lambda *shape, dtype=torch.float16, device="cuda": torch.zeros(shape, dtype=dtype, device=device)  # noqa: E731
    for bad in (t(56, 16, device="cpu"), t(56, 16, dtype=torch.bfloat16), t(55, 16), t(16, 56).T):
        with pytest.raises(AssertionError):
            fs.fs_spmm(fmt, bad)
        with pytest.raises(AssertionError):
            fs.fs_sddmm(fmt, t(40, 16), bad)
        with pytest.raises(AssertionError):
            fs.fs_attention(fmt, t(40, 16), t(56, 16), bad)
    for call in (lambda: fs.fs_spmm(fmt, t(56, 12)), lambda: fs.fs_sddmm(fmt, t(40, 12), t(56, 12)),
                 lambda: fs.fs_attention(fmt, t(40, 16), t(56, 16), t(56, 12))):
        with pytest.raises(fs.FsError) as e:
            call()
        assert e.value.code == 1
    for call in (lambda: fs.fs_edge_softmax(fmt, t(3)), lambda: fs.fs_csr_to_blk(fmt, t(3)), lambda: fs.fs_gather16(t(3), t(3))):
        with pytest.raises(AssertionError):
            call()


def test_value_arrays_are_checked_before_they_are_read(fs):  # noqa: F811
    """fs_blk_to_csr and the ``vals`` of the SpMM calls: too short, on the host, strided, of another type -- refused by
    the call with or without its result given; longer arrays and raw bits stay accepted."""
    A = random_csr(40, 56, 0.2, "f16", seed=7)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, 40, 56)
    n, own = fmt.V * fmt.nvec, fmt.vals_blk_t()
    t = lambda n, dtype=torch.float16, device="cuda": torch.zeros(n, dtype=dtype, device=device)  # noqa: E731
    B, C = torch.ones((56, 16), dtype=torch.float16, device="cuda"), t((40, 16))
    calls = {"fs_blk_to_csr": lambda v: fs.fs_blk_to_csr(fmt, v), "out": lambda v: fs.fs_blk_to_csr(fmt, v, out=t(fmt.nnz)),
             "fs_spmm": lambda v: fs.fs_spmm(fmt, B, vals=v), "fs_spmm out": lambda v: fs.fs_spmm(fmt, B, vals=v, out=C),
             "bind_spmm": lambda v: fs.bind_spmm(fmt, B, C, vals=v)(), "fs_spmm_static": lambda v: fs.fs_spmm_static(fmt, B, C, vals=v)}
    for name, call in calls.items():
        for bad in (t(n - 1), t(n, device="cpu"), t(2 * n)[::2], t(n, torch.float32)):
            with pytest.raises(AssertionError):
                call(bad)
        if "csr" not in name and name != "out":
            with pytest.raises(AssertionError):
                call(t(n, torch.bfloat16))
        want = call(own).clone()
        for good in (torch.cat([own, t(8)]), own.view(torch.int16)):
            same(call(good).view(torch.float16), want)
    for bad in (t(fmt.nnz - 1), t(fmt.nnz, device="cpu"), t(2 * fmt.nnz)[::2], t(fmt.nnz, torch.float32)):
        with pytest.raises(AssertionError):
            fs.fs_blk_to_csr(fmt, own, out=bad)
    for bad in (t(n, device="cpu"), t(n, torch.float32)):
        with pytest.raises(AssertionError):
            fs.fs_csr_to_blk(fmt, va, out=bad)


@pytest.mark.parametrize("call", ["spmm", "spmm out", "bind_spmm", "spmm_packed", "attention", "attention out", "sddmm_spmm", "softmax",
                                  "softmax out", "softmax_backward", "softmax_backward out", "transpose", "convert"])
@pytest.mark.parametrize("external", [False, True])
def test_temporary_memory_belongs_to_the_stream_of_the_kernels(fs, call, external):  # noqa: F811
    """What a call allocates and gives back comes from the memory of ``stream``, not from the current stream's, whose next
    allocation could have it while the kernels are still running."""
    A = random_csr(64, 900, 0.5, "f16", seed=7)
    rp, ci, va = upload_csr(A)
    fmt = fs.fs_convert(rp, ci, va, 64, 900, chunk=64)
    assert fmt.n_split_items > 0  # a workspace is needed
    X, Y, B = (torch.ones((r, c), dtype=torch.float16, device="cuda") for r, c in ((64, 40), (900, 40), (900, 48)))
    out, P, packed = X.new_empty(64, 48), fmt.vals_blk_t().clone(), fs.fs_pack_values(fmt)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()

    class Handle:  # what other frameworks' streams look like
        cuda_stream = side.cuda_stream
    stream = Handle() if external else side
    calls = {
        "spmm": lambda s: fs.fs_spmm(fmt, B, stream=s), "spmm out": lambda s: fs.fs_spmm(fmt, B, out=out, stream=s),
        "bind_spmm": lambda s: fs.bind_spmm(fmt, B, out, stream=s)(), "spmm_packed": lambda s: fs.fs_spmm_packed(fmt, packed, B, stream=s),
        "attention": lambda s: fs.fs_attention(fmt, X, Y, B, stream=s), "attention out": lambda s: fs.fs_attention(fmt, X, Y, B, out=out, stream=s),
        "sddmm_spmm": lambda s: fs.fs_sddmm_spmm(fmt, X, Y, B, stream=s), "softmax": lambda s: fs.fs_edge_softmax(fmt, P, stream=s),
        "softmax out": lambda s: fs.fs_edge_softmax(fmt, P, out=torch.empty_like(P), stream=s),
        "softmax_backward": lambda s: fs.fs_edge_softmax_backward(fmt, P, P, stream=s),
        "softmax_backward out": lambda s: fs.fs_edge_softmax_backward(fmt, P, P, out=torch.empty_like(P), stream=s),
        "transpose": lambda s: fs.fs_csr_transpose(rp, ci, 64, 900, stream=s)[2].view(torch.int16),
        "convert": lambda s: fs.fs_convert(rp, ci, va, 64, 900, chunk=64, stream=s).vals_blk_t(),
    }
    want = calls[call](None).clone()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()  # nothing is left of what earlier tests allocated on this stream

    def held():
        return sum(g["total_size"] for g in torch.cuda.memory_snapshot() if g["stream"] == side.cuda_stream)
    assert held() == 0
    got = calls[call](stream)
    assert held() > 0
    same(got, want)
