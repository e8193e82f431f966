"""GPU parity of the edge softmax (through the C ABI) against the CPU oracle, and the attention chain
SDDMM -> softmax -> SpMM.  Bar: |gpu - ref| <= 1e-2 * ref (+ the output type's subnormal floor); positions
outside the pattern are +0.0 bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import BAR, from_dev_bits, scaled_error, to_dev, upload_csr
from workloads import Csr, bits_to_f64, csr_from_coo, dense, make_config, random_csr, round_to_bits, stream

pytestmark = pytest.mark.gpu
TOL = 1e-2


@pytest.fixture(scope="module")
def fs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2412_11007_amd as fs
    fs.load_library()  # raises if the HIP library is missing: there is no fallback
    return fs


def convert(fs, A, V=8, chunk=0):
    rp, ci, va = upload_csr(A)
    return fs.fs_convert(rp, ci, va, A.M, A.K, torch_dtype=va.dtype, V=V, chunk=chunk)


def check(fs, A, fmt, out_blk, scale):
    """Relative error of the stored positions against the oracle; everything else must be +0.0."""
    ref = oracle.edge_softmax(A.M, A.rowptr, A.vals, A.dtype, scale=scale)
    got_csr = from_dev_bits(fs.fs_blk_to_csr(fmt, out_blk))
    err = scaled_error(got_csr, ref, ref, A.dtype)  # S = ref: plain relative error
    blk = from_dev_bits(out_blk).copy()
    blk[fmt.csr_to_slot_t().cpu().numpy()] = 0
    assert not blk.any(), "non-zero bits outside the pattern"
    # rows sum to one (within the rounding of deg terms)
    sums = np.bincount(np.repeat(np.arange(A.M), np.diff(A.rowptr)), weights=bits_to_f64(got_csr, A.dtype), minlength=A.M)
    deg = np.diff(A.rowptr)
    assert np.abs(sums[deg > 0] - 1).max() <= (2.0 ** -8 if A.dtype == "bf16" else 2.0 ** -10)
    return err


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [4, 8, 16])
@pytest.mark.parametrize("scale,chunk,inplace", [(1.0, 0, False), (0.25, 32, True), (-3.0, 64, False)])
def test_softmax_small(fs, V, dtype, scale, chunk, inplace):
    A = random_csr(203, 150, 0.15, dtype, seed=V + int(scale * 8) + 40, empty_rows=0.2)
    fmt = convert(fs, A, V, chunk)
    vals = fmt.vals_blk_t().clone()
    out = fs.fs_edge_softmax(fmt, vals, out=vals if inplace else None, scale=scale)
    assert check(fs, A, fmt, out, scale) <= BAR[A.dtype]


@pytest.mark.parametrize("V,chunk", [(8, 0), (8, 32), (16, 96), (4, 64)])
def test_softmax_windows_cut_across_items(fs, V, chunk):
    """A few very long rows: their windows span many work items, so the statistics are merged from parts."""
    rng = np.random.default_rng(V + chunk)
    M, K = 70, 6000
    rows, cols = [], []
    for i in range(M):
        deg = 3000 if i in (3, 41) else (900 if i == 20 else int(rng.integers(0, 12)))
        cs = rng.choice(K, size=deg, replace=False)
        rows.append(np.full(deg, i)); cols.append(cs)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    A = csr_from_coo(M, K, rows, cols, "n01", "f16", rng)
    fmt = convert(fs, A, V, chunk)
    assert fmt.n_split_windows > 0
    out = fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=1.5)
    assert check(fs, A, fmt, out, 1.5) <= BAR[A.dtype]
    again = fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=1.5)
    assert np.array_equal(from_dev_bits(out), from_dev_bits(again))  # deterministic
    # a workspace smaller than the parts need is refused before anything is launched
    import torch
    need = fs.fs_edge_softmax_workspace_bytes(fmt)
    assert need == fmt.n_split_items * 2 * V * 4
    with pytest.raises(fs.FsError) as e:
        fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), work=torch.empty(need - 4, dtype=torch.uint8, device="cuda"))
    assert e.value.code == 4


def test_softmax_special_rows_and_arguments(fs):
    import torch
    # uniform scores -> 1/deg exactly where 1/deg is representable; a single entry -> 1; an empty matrix
    rowptr = np.array([0, 4, 4, 5, 13], dtype=np.int32)
    colidx = np.array([0, 5, 9, 30, 2, 1, 2, 3, 4, 5, 6, 7, 8], dtype=np.int32)
    A = Csr(4, 40, rowptr, colidx, round_to_bits(np.full(13, 0.75, dtype=np.float32), "f16"), "f16")
    fmt = convert(fs, A)
    got = bits_to_f64(from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=2.0))), "f16")
    assert np.array_equal(got, np.array([0.25] * 4 + [1.0] + [0.125] * 8))
    E = Csr(16, 16, np.zeros(17, dtype=np.int32), np.zeros(0, dtype=np.int32), np.zeros(0, dtype=np.uint16), "f16")
    fe = convert(fs, E)
    fs.fs_edge_softmax(fe, torch.empty(0, dtype=torch.float16, device="cuda"))
    # argument checks
    with pytest.raises(fs.FsError) as e:
        fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=float("nan"))
    assert e.value.code == 1
    with pytest.raises(fs.FsError) as e:
        fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=float("inf"))
    assert e.value.code == 1


@pytest.mark.parametrize("V", [4, 8])
def test_softmax_keeps_bf16_subnormal_probabilities(fs, V):
    """A peaked bf16 row: probabilities between 2^-133 and 2^-126 are subnormal in bf16 AND in fp32, the
    range where a fast fp32 exponential returns zero.  The kernel must still deliver them."""
    M, K = 9, 70
    rows = np.repeat(np.arange(M), 40)
    cols = np.tile(np.arange(40), M)
    A = csr_from_coo(M, K, rows, cols, "u01", "bf16", np.random.default_rng(0))
    # scores 0, -86, -86.5, ... -92: exp(-88) = 6e-39 and exp(-91.5) = 2e-40 are both bf16 subnormals
    row_scores = np.concatenate([[0.0], -86.0 - 0.5 * np.arange(13), -20.0 - np.arange(26)]).astype(np.float32)
    A.vals = np.tile(round_to_bits(row_scores, "bf16"), M)
    fmt = convert(fs, A, V)
    out = fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=1.0)
    got = bits_to_f64(from_dev_bits(fs.fs_blk_to_csr(fmt, out)), "bf16")
    ref = oracle.edge_softmax(A.M, A.rowptr, A.vals, "bf16", scale=1.0)
    tiny = (ref > 0) & (ref < 2.0 ** -126)
    assert tiny.sum() >= 5 * M and (got[tiny] > 0).all()
    assert check(fs, A, fmt, out, 1.0) <= BAR[A.dtype]


@pytest.mark.parametrize("name", ["cfg2_rmat16", "cfg5_lognormal"])
def test_attention_chain_full_configs(fs, name):
    """SDDMM scores -> edge softmax -> SpMM on the GPU, each stage against the oracle fed the GPU's own
    16-bit input of that stage, and the whole chain against an independent oracle chain."""
    c = make_config(name)
    A = c["A"]
    X, Y = c["sddmm"]
    H = c["chain"] if "chain" in c else c["spmm"][0]
    d = X.shape[1]
    scale = 1.0 / np.sqrt(d)
    fmt = convert(fs, A)
    scores = fs.fs_sddmm(fmt, to_dev(X.bits, "f16"), to_dev(Y.bits, "f16"))
    att = fs.fs_edge_softmax(fmt, scores, scale=scale)
    C = from_dev_bits(fs.fs_spmm(fmt, to_dev(H.bits, "f16"), vals=att))
    # stage 2 alone
    gpu_scores = from_dev_bits(fs.fs_blk_to_csr(fmt, scores))
    As = Csr(A.M, A.K, A.rowptr, A.colidx, gpu_scores, "f16")
    err_sm = check(fs, As, fmt, att, scale)
    # stage 3 alone
    gpu_att = from_dev_bits(fs.fs_blk_to_csr(fmt, att))
    ref, S = oracle.spmm(A.M, A.K, A.rowptr, A.colidx, gpu_att, H.bits, "f16")
    err_spmm = scaled_error(C, ref, S, "f16")
    # whole chain, oracle only
    sref, _ = oracle.sddmm(A.M, A.K, A.rowptr, A.colidx, X.bits, Y.bits, "f16")
    aref = oracle.edge_softmax(A.M, A.rowptr, oracle.round_f64_to_bits(sref, "f16"), "f16", scale=scale)
    ref2, S2 = oracle.spmm(A.M, A.K, A.rowptr, A.colidx, oracle.round_f64_to_bits(aref, "f16"), H.bits, "f16")
    err_chain = scaled_error(C, ref2, S2, "f16")
    print("\n%s attention chain: softmax %.3e, spmm %.3e, whole chain %.3e" % (name, err_sm, err_spmm, err_chain))
    assert err_sm <= TOL and err_spmm <= TOL and err_chain <= TOL


# ---------------------------------------------------------------- gradient of the edge softmax
def hub_csr(M, K, dtype, seed):
    """A few rows with thousands of entries (windows cut into many parts) among short and empty ones."""
    rng = np.random.default_rng(seed)
    rows, cols = [], []
    for i in range(M):
        deg = 3000 if i in (3, M - 2) else (900 if i == M // 2 else int(rng.integers(0, 12)))
        rows.append(np.full(deg, i)); cols.append(rng.choice(K, size=deg, replace=False))
    return csr_from_coo(M, K, np.concatenate(rows), np.concatenate(cols), "n01", dtype, rng)


def run_backward(fs, A, fmt, p_bits, g_bits, scale, inplace=False):
    """GPU gradient for probabilities / incoming gradients given in CSR order; returns (CSR-order bits, blocked bits)."""
    p_blk = fs.fs_csr_to_blk(fmt, to_dev(p_bits, A.dtype))
    g_blk = fs.fs_csr_to_blk(fmt, to_dev(g_bits, A.dtype))
    out = fs.fs_edge_softmax_backward(fmt, p_blk, g_blk, out=p_blk if inplace else None, scale=scale)
    got_csr = from_dev_bits(fs.fs_blk_to_csr(fmt, out))
    blk = from_dev_bits(out).copy()
    blk[fmt.csr_to_slot_t().cpu().numpy()] = 0
    assert not blk.any(), "non-zero bits outside the pattern"
    return got_csr


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [4, 8, 16])
@pytest.mark.parametrize("scale,chunk,inplace", [(1.0, 0, False), (0.25, 32, True), (-3.0, 64, False)])
def test_softmax_backward_small(fs, V, dtype, scale, chunk, inplace):
    """Probabilities from the GPU's own forward call (so they are what a training step would hold),
    a random incoming gradient; against the oracle on the same 16-bit inputs."""
    A = random_csr(203, 150, 0.15, dtype, seed=V + int(scale * 8) + 70, empty_rows=0.2)
    fmt = convert(fs, A, V, chunk)
    p_bits = from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=scale)))
    g_bits = round_to_bits(stream(V, 96, 1).normal(size=A.nnz).astype(np.float32), dtype)
    got = run_backward(fs, A, fmt, p_bits, g_bits, scale, inplace)
    ref, S = oracle.edge_softmax_backward(A.M, A.rowptr, p_bits, g_bits, dtype, scale=scale)
    assert scaled_error(got, ref, S, dtype) <= BAR[dtype]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V,chunk", [(8, 0), (8, 32), (16, 96), (4, 64)])
def test_softmax_backward_windows_cut_across_items(fs, V, chunk, dtype):
    """Rows of thousands of entries: the row sums of p * g are merged from the parts' partial sums."""
    A = hub_csr(70, 6000, dtype, seed=V + chunk)
    fmt = convert(fs, A, V, chunk)
    assert fmt.n_split_windows > 0
    p_bits = from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_edge_softmax(fmt, fmt.vals_blk_t(), scale=1.5)))
    g_bits = round_to_bits(stream(V, 96, 2).normal(size=A.nnz).astype(np.float32), dtype)
    got = run_backward(fs, A, fmt, p_bits, g_bits, 1.5)
    ref, S = oracle.edge_softmax_backward(A.M, A.rowptr, p_bits, g_bits, dtype, scale=1.5)
    assert scaled_error(got, ref, S, dtype) <= BAR[dtype]
    assert np.array_equal(got, run_backward(fs, A, fmt, p_bits, g_bits, 1.5))  # deterministic
    import torch
    need = fs.fs_edge_softmax_workspace_bytes(fmt)
    blk = fs.fs_csr_to_blk(fmt, to_dev(p_bits, dtype))
    with pytest.raises(fs.FsError) as e:
        fs.fs_edge_softmax_backward(fmt, blk, blk, work=torch.empty(need - 4, dtype=torch.uint8, device="cuda"))
    assert e.value.code == 4


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [4, 8, 16])
def test_softmax_backward_bit_exact(fs, V, dtype):
    """Probabilities k/64 and gradients that are multiples of 1/4: every product and every partial sum is
    exact in fp32 whatever the order, so the only rounding on either side is the one to the 16-bit type --
    GPU bits == oracle bits, hub rows cut into dozens of parts included."""
    A = hub_csr(70, 6000, dtype, seed=V + 5)
    rng = stream(V, 96, 3)
    deg = np.diff(A.rowptr)
    # p = k/64 with small k (the values need not sum to one: the kernel computes the formula on what it is given)
    p = rng.integers(0, 5, size=A.nnz).astype(np.float32) / 64.0
    g = rng.integers(-8, 9, size=A.nnz).astype(np.float32) / 4.0
    p_bits, g_bits = round_to_bits(p, dtype), round_to_bits(g, dtype)
    fmt = convert(fs, A, V, chunk=64)
    assert fmt.n_split_windows >= 3
    got = run_backward(fs, A, fmt, p_bits, g_bits, 0.5)
    ref, _ = oracle.edge_softmax_backward(A.M, A.rowptr, p_bits, g_bits, dtype, scale=0.5)
    # p g and the row sums are multiples of 2^-8 below 2^9 (17 bits), g - dot as well; times p = k/64 with k <= 4
    # and times the scale 1/2 that makes multiples of 2^-15 of at most 20 bits: exact in fp32 on the GPU as in fp64 here
    assert np.array_equal(ref * 2.0 ** 15, np.rint(ref * 2.0 ** 15)) and np.abs(ref).max() < 2.0 ** 5
    want = oracle.round_f64_to_bits(ref, dtype)
    bad = np.nonzero(got != want)[0]
    assert bad.size == 0, "%d of %d differ, first at %d: gpu 0x%04x, expected 0x%04x (degree %d)" % (
        bad.size, got.size, bad[0], got[bad[0]], want[bad[0]], deg[np.searchsorted(A.rowptr, bad[0], side="right") - 1])


def test_softmax_backward_arguments_and_empty(fs):
    import torch
    A = random_csr(40, 30, 0.2, "f16", seed=3)
    fmt = convert(fs, A)
    v = fmt.vals_blk_t()
    for bad in (float("nan"), float("inf")):
        with pytest.raises(fs.FsError) as e:
            fs.fs_edge_softmax_backward(fmt, v, v, scale=bad)
        assert e.value.code == 1
    E = Csr(16, 16, np.zeros(17, dtype=np.int32), np.zeros(0, dtype=np.int32), np.zeros(0, dtype=np.uint16), "f16")
    fe = convert(fs, E)
    z = torch.empty(0, dtype=torch.float16, device="cuda")
    fs.fs_edge_softmax_backward(fe, z, z)


def test_attention_backward_chain_matches_finite_differences(fs):
    """The calls compose into the backward pass of out = softmax_rows(scale * X Y^T at A's pattern) * H:
        P = fs_edge_softmax(fs_sddmm(X, Y)),  G = fs_sddmm(dOut, H),  dS = fs_edge_softmax_backward(P, G),
        dX = fs_spmm(values dS, Y),  dY = fs_spmm(A^T, values dS, X),  dH = fs_spmm(A^T, values P, dOut).
    Checked against central differences of the fp64 attention oracle for L = sum(out * dOut); the chain rounds
    P, G and dS to 16 bits on the way, hence the loose bar."""
    M, K, d, N, scale = 24, 40, 16, 16, 0.25
    A = random_csr(M, K, 0.2, "f16", seed=12, empty_rows=0.1)
    rng = np.random.default_rng(4)
    Xf = (np.round(rng.normal(size=(M, d)) * 8) / 8).astype(np.float32)
    Yf = (np.round(rng.normal(size=(K, d)) * 8) / 8).astype(np.float32)
    Hf = (np.round(rng.normal(size=(K, N)) * 8) / 8).astype(np.float32)
    Rf = (np.round(rng.normal(size=(M, N)) * 8) / 8).astype(np.float32)
    Xb, Yb, Hb, Rb = (round_to_bits(a, "f16") for a in (Xf, Yf, Hf, Rf))
    fmt = convert(fs, A)
    X, Y, H, R = (to_dev(b, "f16") for b in (Xb, Yb, Hb, Rb))
    P = fs.fs_edge_softmax(fmt, fs.fs_sddmm(fmt, X, Y), scale=scale)
    G = fs.fs_sddmm(fmt, R, H)
    dS = fs.fs_edge_softmax_backward(fmt, P, G, scale=scale)
    dX = bits_to_f64(from_dev_bits(fs.fs_spmm(fmt, Y, vals=dS)), "f16")

    def loss(Xv):
        out, _ = oracle.attention(M, K, A.rowptr, A.colidx, round_to_bits(Xv.astype(np.float32), "f16"), Yb, Hb, "f16", scale)
        return float((out * Rf.astype(np.float64)).sum())

    # X moves on the fp16 grid: steps of 2^-6 around values that are multiples of 1/8 stay exactly representable
    h = 2.0 ** -6
    fd = np.zeros((M, d))
    for i in range(M):
        for t in range(d):
            E = np.zeros((M, d)); E[i, t] = h
            fd[i, t] = (loss(Xf + E) - loss(Xf - E)) / (2 * h)
    scale_of = np.abs(fd).max()
    assert np.abs(dX - fd).max() <= 2e-2 * scale_of, (np.abs(dX - fd).max(), scale_of)

    # dY = dS^T X and dH = P^T dOut: the same products on the converted transpose, values carried over by the
    # permutation fs_csr_transpose returns
    import torch
    rp, ci, _ = upload_csr(A)
    rp_t, ci_t, perm = fs.fs_csr_transpose(rp, ci, M, K)
    P_t = fs.fs_gather16(fs.fs_blk_to_csr(fmt, P), perm)
    fmt_t = fs.fs_convert(rp_t, ci_t, P_t, K, M, torch_dtype=torch.float16)
    dH = bits_to_f64(from_dev_bits(fs.fs_spmm(fmt_t, R)), "f16")
    dS_t = fs.fs_csr_to_blk(fmt_t, fs.fs_gather16(fs.fs_blk_to_csr(fmt, dS), perm))
    dY = bits_to_f64(from_dev_bits(fs.fs_spmm(fmt_t, X, vals=dS_t)), "f16")

    def loss_yh(Yv, Hv):
        out, _ = oracle.attention(M, K, A.rowptr, A.colidx, Xb, round_to_bits(Yv.astype(np.float32), "f16"),
                                  round_to_bits(Hv.astype(np.float32), "f16"), "f16", scale)
        return float((out * Rf.astype(np.float64)).sum())

    fdY, fdH = np.zeros((K, d)), np.zeros((K, N))
    for k in range(K):
        for t in range(d):
            E = np.zeros((K, d)); E[k, t] = h
            fdY[k, t] = (loss_yh(Yf + E, Hf) - loss_yh(Yf - E, Hf)) / (2 * h)
        for t in range(N):
            E = np.zeros((K, N)); E[k, t] = h
            fdH[k, t] = (loss_yh(Yf, Hf + E) - loss_yh(Yf, Hf - E)) / (2 * h)
    assert np.abs(dY - fdY).max() <= 2e-2 * np.abs(fdY).max(), (np.abs(dY - fdY).max(), np.abs(fdY).max())
    assert np.abs(dH - fdH).max() <= 2e-2 * np.abs(fdH).max(), (np.abs(dH - fdH).max(), np.abs(fdH).max())


@pytest.mark.parametrize("V,chunk", [(4, 0), (8, 0), (8, 32), (16, 64)])
def test_softmax_of_a_format_without_row_occupancies(fs, V, chunk):
    """A format that somebody put together with the vectors' masks alone: the same bits as with the rows' occupancies."""
    import torch
    M, K, dtype = 180, 5000, "f16"
    A = hub_csr(M, K, dtype, 77 + V)
    fmt = convert(fs, A, V, chunk)
    assert fmt.n_split_items > 0
    vals, g = fmt.vals_blk_t(), torch.randn(V * fmt.nvec, generator=torch.Generator("cuda").manual_seed(V), device="cuda").half()
    p = fs.fs_edge_softmax(fmt, vals, scale=0.5)
    d = fs.fs_edge_softmax_backward(fmt, p, g, scale=0.5)
    bare = fs.FsFormat(type(fmt.c).from_buffer_copy(fmt.c), fmt.arena, fmt.torch_dtype)
    bare.c.blk_row_bits = None
    for out in (torch.full_like(vals, 3.0), None):
        assert torch.equal(fs.fs_edge_softmax(bare, vals, out=out, scale=0.5).view(torch.int16), p.view(torch.int16))
    assert torch.equal(fs.fs_edge_softmax_backward(bare, p, g, scale=0.5).view(torch.int16), d.view(torch.int16))


@pytest.mark.parametrize("V", [4, 8, 16])
@pytest.mark.parametrize("offset", [0, 1, 2, 3, 5])
def test_softmax_arrays_begin_on_any_element(fs, V, offset):
    """Value arrays that are part of a larger buffer, and with four rows blocks that begin eight bytes past a line: sixteen bytes
    are moved at a time wherever they lie, and nothing beside the array is written."""
    import torch
    fmt = convert(fs, random_csr(303, 170, 0.2, "f16", seed=V, empty_rows=0.1), V, 0)
    n = V * fmt.nvec
    gen = torch.Generator("cuda").manual_seed(offset)
    vals, g = (torch.randn(n, generator=gen, device="cuda").half() for _ in range(2))
    p = fs.fs_edge_softmax(fmt, vals)
    d = fs.fs_edge_softmax_backward(fmt, p, g)

    def moved(t):
        buf = torch.full((n + 16,), 7.0, dtype=torch.float16, device="cuda")
        buf[offset:offset + n] = t
        return buf

    a, b, out = moved(vals), moved(g), moved(torch.zeros_like(vals))
    fs.fs_edge_softmax(fmt, a[offset:offset + n], out=out[offset:offset + n])
    assert torch.equal(out.view(torch.int16), moved(p).view(torch.int16))
    fs.fs_edge_softmax(fmt, a[offset:offset + n], out=a[offset:offset + n])
    assert torch.equal(a.view(torch.int16), moved(p).view(torch.int16))
    fs.fs_edge_softmax_backward(fmt, a[offset:offset + n], b[offset:offset + n], out=b[offset:offset + n])
    assert torch.equal(b.view(torch.int16), moved(d).view(torch.int16))


def ragged_windows(V, dtype, seed, large):
    """Windows of 0 to 10 blocks in every order, the last block of most of them narrow, and a few long enough to be cut; `large` windows
    have scores so far apart that the exponential needs care (a range of +-60 after scaling by one), beside others that have not."""
    rng = np.random.default_rng(seed)
    K, blocks = 6000, np.concatenate([np.repeat(np.arange(11), 9), [14, 20, 60, 13]])
    rng.shuffle(blocks)
    rows, cols, span = [], [], []
    for w, n_b in enumerate(blocks):
        n = 0 if n_b == 0 else 32 * (n_b - 1) + int(rng.choice([1, 7, 8, 9, 31, 32]))
        c = rng.choice(K, size=n, replace=False)
        r = np.concatenate([rng.integers(0, V, n), rng.integers(0, V, n // 3)])  # every vector in one or two rows
        rows.append(w * V + r)
        cols.append(np.concatenate([c, c[:n // 3]]))
        span.append(np.full(r.size, 60.0 if large and w % 3 == 0 else 1.0))
    rows, cols, span = (np.concatenate(x) for x in (rows, cols, span))
    keep = np.unique(rows * K + cols, return_index=True)[1]  # in CSR order
    A = csr_from_coo(len(blocks) * V, K, rows[keep], cols[keep], "n01", dtype, rng)
    A.vals[:] = round_to_bits((rng.uniform(-1, 1, keep.size) * span[keep]).astype(np.float32), dtype)
    return A


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [4, 8, 16])
@pytest.mark.parametrize("chunk,large", [(0, False), (0, True), (128, True), (256, False), (1024, True)])
def test_softmax_items_around_a_register_load(fs, V, dtype, chunk, large):
    """Items with whole windows and parts of cut ones, as long as one load of blocks holds, shorter and longer: both walks and both
    exponentials, in place as well as not."""
    import torch
    A = ragged_windows(V, dtype, V + chunk, large)
    fmt = convert(fs, A, V, chunk)
    n = fmt.items_t()[:, 1].cpu().numpy()
    for at in (4, 8) if chunk >= 256 else (4,):  # (shorter parts make no items of eight)
        assert (n < at).any() and (n == at).any() and (n > at).any(), np.bincount(n)
    assert fmt.n_split_items > 0
    vals = fmt.vals_blk_t().clone()
    out = fs.fs_edge_softmax(fmt, vals)
    assert check(fs, A, fmt, out, 1.0) <= BAR[dtype]
    assert torch.equal(fs.fs_edge_softmax(fmt, vals, out=vals).view(torch.int16), out.view(torch.int16))

    # the gradient, against the definition in 64 bits on the same probabilities
    p_bits = from_dev_bits(fs.fs_blk_to_csr(fmt, out))
    g_bits = A.vals
    got = bits_to_f64(run_backward(fs, A, fmt, p_bits, g_bits, 0.5, inplace=True), dtype)
    p, g = bits_to_f64(p_bits, dtype), bits_to_f64(g_bits, dtype)
    row = np.repeat(np.arange(A.M), np.diff(A.rowptr))
    dot, size = (np.bincount(row, weights=x, minlength=A.M)[row] for x in (p * g, np.abs(p * g)))
    # one rounding of the result, and fp32 sums whose terms are no larger than `size`: 2^-20 holds some hundred of them
    bound = 0.5 * p * (np.abs(g - dot) * BAR[dtype] + (size + np.abs(g)) * 2.0 ** -20) + {"f16": 2.0 ** -24, "bf16": 2.0 ** -133}[dtype]
    assert (np.abs(got - 0.5 * p * (g - dot)) <= bound).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("V", [4, 8, 16])
def test_softmax_of_scores_that_are_no_numbers(fs, V, dtype):
    """A NaN makes its row zeros and touches no other, however the work list is cut and whatever else its lane holds."""
    import torch
    A = ragged_windows(V, dtype, 5 + V, False)
    rng = np.random.default_rng(V)
    row = np.repeat(np.arange(A.M), np.diff(A.rowptr))
    bad = rng.choice(A.nnz, 60, replace=False)
    fine = ~np.isin(row, row[bad])
    nan = A.vals.copy()
    nan[bad] = 0x7E00 if dtype == "f16" else 0x7FC0
    for chunk in (0, 32, 256, 1024):
        fmt = convert(fs, A, V, chunk)
        want = from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_edge_softmax(fmt, fmt.vals_blk_t())))
        got = from_dev_bits(fs.fs_blk_to_csr(fmt, fs.fs_edge_softmax(fmt, fs.fs_csr_to_blk(fmt, to_dev(nan, dtype)))))
        assert np.array_equal(got[fine], want[fine]) and not got[~fine].any(), chunk
