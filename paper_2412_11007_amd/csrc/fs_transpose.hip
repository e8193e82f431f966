// CSR of the transposed matrix, entirely on the GPU and without a host synchronisation.
//
// Training a GNN layer (the paper's Section 4.4 workloads) needs A^T * dC in the backward pass of
// C = A * B.  This library computes it with the same kernels on a second converted format, that of
// A^T; this file produces the CSR that conversion starts from, plus the permutation that carries
// per-entry values (edge weights, attention coefficients) from A's order into A^T's.
//
// The stored entries of A, taken in CSR order, are sorted by (row, column).  A STABLE sort of them by
// column alone therefore leaves them sorted by (column, row): the CSR order of A^T.  The sort is the
// least-significant-digit radix sort of fs_sort.h on the column index.  Up to 2^20 columns it takes two passes, and a word
// has room for a column's upper digit and the row, which then travel together: the last pass leaves the column indices of
// A^T, with no gather through the permutation, and the counts of both passes tell where A^T's rows start (5.3 M entries,
// 18 bits: 320 -> 151 us with the values, of which a gather of rows was 70 and the table it read 16).
// No atomics touch global memory and the result does not depend on scheduling.
#include <algorithm>
#include <type_traits>

#include "fs_common.h"
#include "fs_rows.h"
#include "fs_scan.h"
#include "fs_sort.h"

namespace {

// rowptr_t[k] = number of entries whose column is below k, k in [0, K].
__global__ void k_rowptr_of_sorted(const int32_t *__restrict__ sorted_cols, int32_t n, int64_t K, int32_t *__restrict__ rowptr_t)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k > K) return;
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (sorted_cols[mid] < k) lo = mid + 1; else hi = mid;
    }
    rowptr_t[k] = lo;
}

// The same from the counts of two passes on low_bits and high_bits column bits (low_bits = 0: of one).  The last pass'
// input is sorted by the low digit, and the low digit `low` starts at first_of[low] of it; so the entries before column
// (high, low) are those the last pass puts before its group's with the digit `high`, and those of that group up to there.  One workgroup
// per low digit, neighbours on one XCD (they write neighbouring pointers).
constexpr int kCountsThreads = 512;
__global__ void __launch_bounds__(kCountsThreads) k_rowptr_of_counts(const uint32_t *__restrict__ words, const int *__restrict__ first_of, const int *__restrict__ start, int ngroup,
                                                          int group, int low_bits, int high_bits, int32_t n, int64_t K, int32_t *__restrict__ rowptr_t)
{
    __shared__ int h[1 << kMaxDigitBits];
    const int lows = 1 << low_bits, per = (lows + 7) / 8;
    const int low = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || low >= lows) return;
    for (int i = threadIdx.x; i < 1 << high_bits; i += kCountsThreads) h[i] = 0;
    __syncthreads();
    const int64_t upto = first_of ? first_of[low] : 0;
    const int g = (int)std::min<int64_t>(upto / group, ngroup - 1);
    constexpr int kAhead = 8;
    for (int64_t i0 = (int64_t)g * group + threadIdx.x; i0 < upto; i0 += kCountsThreads * kAhead) {
        uint32_t word[kAhead];
#pragma unroll
        for (int r = 0; r < kAhead; r++) word[r] = words[std::min(i0 + r * kCountsThreads, upto - 1)];
#pragma unroll
        for (int r = 0; r < kAhead; r++)
            if (i0 + r * kCountsThreads < upto) atomicAdd(&h[word[r] & ((1u << high_bits) - 1)], 1);
    }
    __syncthreads();
    for (int high = threadIdx.x; high < 1 << high_bits; high += kCountsThreads) {
        const int64_t k = (int64_t)high << low_bits | low;
        if (k < K) rowptr_t[k] = start[(int64_t)high * ngroup + g] + h[high];
    }
    if (low == 0 && threadIdx.x == 0) rowptr_t[K] = n;
}

// row_of[p] = the row of A that stores entry p: the last r with rowptr[r] <= p.
__global__ void __launch_bounds__(kEntriesPerGroup) k_row_of_entry(const int32_t *__restrict__ rowptr, int64_t n,
                                                                    const int32_t *__restrict__ group_rows,
                                                                    int32_t *__restrict__ row_of)
{
    __shared__ int32_t sh_ptr[kEntriesPerGroup];
    const int64_t p = (int64_t)blockIdx.x * kEntriesPerGroup + threadIdx.x;
    const int64_t r = group_row_of(rowptr, n, p, group_rows, sh_ptr);
    if (r >= 0) row_of[p] = (int32_t)r;
}

// colidx_t[i] = row_of[perm[i]]
__global__ void k_gather_i32(const int32_t *__restrict__ src, const int32_t *__restrict__ idx, int64_t n, int32_t *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[idx[i]];
}

__global__ void k_fill_i32(int32_t *__restrict__ dst, int64_t n, int32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = v;
}

__global__ void k_gather16(const uint16_t *__restrict__ src, const int32_t *__restrict__ idx, int64_t n, uint16_t *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[idx[i]];
}

// The same where there are many indices.  If a source is more than an XCD's L2 holds, nearly every element is a missed line
// (5.3 M elements through a random permutation: 61 us, 24 from a source of 2 MB).  A workgroup then sorts its 4096 indices by
// band of the source (2^shift elements, the last band open) in LDS and loads in that order, one load in flight per lane, so
// that all wavefronts pass through the bands at about one pace and a band is in every L2 while it is read: 40 us.  (With all
// sixteen loads issued at once the oldest wavefronts run ahead through all bands, and nothing is gained.)  From the first workgroup
// on that has to wait for a place on the chip (8.4 M elements) the pace is lost, bit by bit.
// PEEK: every wavefront first looks at 64 of its indices; where they, and those of the workgroup's other wavefronts, lie close
// together (a mesh' permutation, a short source, a copy), all are loaded as they come.  Permutation of a 1024^2 mesh, 5.2 M: one
// element a thread 13.2 us, sorted 16.6, as they come 10.9; 3 M indices into 512 KB 13.5, 16.9 and 14.6.
constexpr int kBands = 16, kBandEach = 16, kBandThreads = 256;
constexpr uint32_t kNear = 5u << 18;  // elements: all indices into 2.5 MB are close together
template <bool PEEK>
__global__ void __launch_bounds__(kBandThreads) __attribute__((amdgpu_waves_per_eu(8))) k_gather16_banded(const uint16_t *__restrict__ src, const int32_t *__restrict__ idx, int64_t n, int shift,
                                                                  uint16_t *__restrict__ dst)
{
    constexpr int kWaves = kBandThreads / 64, kAll = kBandThreads * kBandEach;
    __shared__ uint32_t stage[kAll];
    __shared__ uint16_t cur[kBands * kWaves];  // band-major
    __shared__ uint2 seen[PEEK ? kWaves : 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t base = (int64_t)blockIdx.x * kAll;
    const int left = (int)std::min<int64_t>(n - base, kAll);
    idx += base;
    dst += base;
    const auto index = [&](int e) -> uint32_t {
        return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(idx) + 4u * (uint32_t)std::min((w * kBandEach + e) * 64 + lane, left - 1));
    };
    const auto element = [&](uint32_t i) -> uint16_t { return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(src) + i * 2u); };
    if constexpr (PEEK) {
        const uint32_t some = index(0), one = (uint32_t)__builtin_amdgcn_readfirstlane((int)some);
        const bool wide = __any(std::max(some, one) - std::min(some, one) > kNear);
        if (lane == 0) seen[w] = make_uint2(wide ? 0u : one, wide ? ~0u : one);
        __syncthreads();
        uint2 range = seen[0];
#pragma unroll
        for (int k = 1; k < kWaves; k++) range = make_uint2(std::min(range.x, seen[k].x), std::max(range.y, seen[k].y));
        if (range.y - range.x <= kNear) {  // the same for the workgroup
            uint32_t at[kBandEach];
            uint16_t v[kBandEach];
#pragma unroll
            for (int e = 0; e < kBandEach; e++) at[e] = index(e);
#pragma unroll
            for (int e = 0; e < kBandEach; e++) v[e] = element(at[e]);
            const uint32_t first = (uint32_t)(w * kBandEach * 64 + lane);
            const int last = left - 1 - (int)first;
#pragma unroll
            for (int e = 0; e < kBandEach; e++)
                if (e * 64 <= last) dst[first + e * 64] = v[e];
            return;
        }
    }
    uint32_t at[kBandEach], slot[kBandEach];
#pragma unroll
    for (int e = 0; e < kBandEach; e++) at[e] = index(e);
    if (lane < kBands) cur[lane * kWaves + w] = 0;
    FS_WAVE_SYNC();
    const uint64_t below = ((uint64_t)1 << lane) - 1;
#pragma unroll
    for (int e = 0; e < kBandEach; e++) {
        asm volatile("" : "+v"(at[e]) : : "memory");  // round by round: run ahead, the ballots would fill the registers
        const uint32_t band = std::min(at[e] >> shift, (uint32_t)kBands - 1);
        uint64_t same = ~0ull;
#pragma unroll
        for (int b = 0; b < 4; b++) {
            const bool bit = (band >> b) & 1;
            const uint64_t set = __ballot(bit);
            same &= bit ? set : ~set;
        }
        const int rank = __popcll(same & below), cnt = __popcll(same);
        const int so_far = cur[band * kWaves + w];
        slot[e] = (uint32_t)(so_far + rank);
        FS_WAVE_SYNC();
        if (rank == cnt - 1) cur[band * kWaves + w] = (uint16_t)(so_far + cnt);
        FS_WAVE_SYNC();
    }
    __syncthreads();
    if (w == 0) {
        const int c = cur[lane];
        cur[lane] = (uint16_t)(wave_inclusive_scan(c) - c);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kBandEach; e++) {
        if (e % 4 == 0) asm volatile("" : "+v"(at[e]), "+v"(at[e + 1]), "+v"(at[e + 2]), "+v"(at[e + 3]) : : "memory");
        slot[e] += cur[std::min(at[e] >> shift, (uint32_t)kBands - 1) * kWaves + w];
        stage[slot[e]] = at[e];
    }
    __syncthreads();
    uint16_t v[kBandEach];
#pragma unroll
    for (int k = 0; k < kBandEach; k++) at[k] = stage[k * kBandThreads + threadIdx.x];
#pragma unroll
    for (int k = 0; k < kBandEach; k++) {
        v[k] = element(at[k]);
        if (k + 1 < kBandEach) asm volatile("" : "+v"(at[k + 1]) : "v"((uint32_t)v[k]));  // the next address only once this element is here
    }
    __syncthreads();
    uint16_t *vals = reinterpret_cast<uint16_t *>(stage);
#pragma unroll
    for (int k = 0; k < kBandEach; k++) vals[k * kBandThreads + threadIdx.x] = v[k];
    __syncthreads();
    int last = left - 1 - (w * kBandEach * 64 + lane);  // this lane's elements 64 e with e * 64 <= last exist
    asm volatile("" : "+v"(last));                      // (compared here, not kept in sixteen registers from the start)
#pragma unroll
    for (int e = 0; e < kBandEach; e++) {
        const int i = (w * kBandEach + e) * 64 + lane;
        if (e * 64 <= last) dst[(uint32_t)i] = vals[slot[e]];
    }
}

inline unsigned grid_of(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

// The passes, and the scratch layout (ints): [keys 0: nnz][keys 1: nnz][payload: nnz][digit counts][scan tmp][first digit's starts]
struct TransposePlan {
    int passes, bits[4];  // digits, low to high
    bool rows;            // rows travel with the keys
    int row_shift;        // of the row in the first pass' output
    size_t key0, key1, val1, hist, tmp, first_of, total_ints;
};
int bits_of(int64_t n)  // of 0 .. n - 1
{
    int b = 0;
    while (b < 31 && ((n - 1) >> b) != 0) b++;
    return b;
}
TransposePlan plan_transpose(int64_t M, int64_t K, int64_t nnz, bool any_size = false)
{
    TransposePlan p;
    // as few passes as digits of ten bits take, evenly wide: 5.3 M entries, 18-bit columns, two passes of nine bits
    const int bits = bits_of(std::max<int64_t>(K, 1));
    p.passes = std::max(1, (bits + kMaxDigitBits - 1) / kMaxDigitBits);
    for (int i = 0, left = bits; i < p.passes; i++) {
        p.bits[i] = (left + p.passes - i - 1) / (p.passes - i);
        left -= p.bits[i];
    }
    p.row_shift = bits - p.bits[0];
    p.rows = p.passes <= 2 && p.row_shift + bits_of(std::max<int64_t>(M, 1)) <= 32;
    // any_size: the room that is asked for, of the widest digits and of the most groups that so many entries or fewer make.  It
    // depends on nnz alone and never goes down as nnz goes up, so that a buffer for the largest of several matrices serves
    // them all.  (A call takes less where it needs less.)
    const int64_t n = std::max<int64_t>(nnz, 1);
    const size_t e = fs_align_up((size_t)nnz, 64), counts = any_size ? (size_t)sort_groups_bound(n) << kMaxDigitBits : (size_t)sort_groups(n) << std::max(8, p.bits[0]);
    size_t o = 0;
    p.key0 = o; o += e;
    p.key1 = o; o += e;  // (not used where rows travel)
    p.val1 = o; o += e;
    p.hist = o; o += fs_align_up(counts + 1, 64);
    p.tmp = o; o += scan_tmp_ints((int64_t)counts);
    p.first_of = o; o += 1 << kMaxDigitBits;
    p.total_ints = o;
    return p;
}

bool sizes_ok(int64_t M, int64_t K, int64_t nnz) { return M >= 0 && K >= 0 && nnz >= 0; }
bool sizes_fit(int64_t M, int64_t K, int64_t nnz)
{
    const int64_t lim = (int64_t)INT32_MAX - 4096;
    return M <= lim && K <= lim && nnz <= lim;
}

}  // namespace

extern "C" fs_status fs_csr_transpose_bytes(int64_t M, int64_t K, int64_t nnz, size_t *scratch_bytes)
{
    if (!scratch_bytes || !sizes_ok(M, K, nnz)) return FS_ERR_INVALID_ARG;
    if (!sizes_fit(M, K, nnz)) return FS_ERR_TOO_LARGE;
    *scratch_bytes = plan_transpose(M, K, nnz, true).total_ints * sizeof(int) + 256;
    return FS_OK;
}

extern "C" fs_status fs_csr_transpose(int64_t M, int64_t K, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                                      int32_t *d_rowptr_t, int32_t *d_colidx_t, int32_t *d_perm, void *d_scratch,
                                      size_t scratch_bytes, void *stream)
{
    if (!sizes_ok(M, K, nnz) || !d_rowptr || !d_rowptr_t) return FS_ERR_INVALID_ARG;
    if (nnz > 0 && (!d_colidx || !d_colidx_t || !d_perm || !d_scratch || M == 0 || K == 0)) return FS_ERR_INVALID_ARG;
    if (!sizes_fit(M, K, nnz)) return FS_ERR_TOO_LARGE;
    hipStream_t st = (hipStream_t)stream;
    if (nnz == 0) {
        k_fill_i32<<<grid_of(K + 1, 256), 256, 0, st>>>(d_rowptr_t, K + 1, 0);
        FS_LAUNCH_CHECK();
        return FS_OK;
    }
    if ((uintptr_t)d_scratch & 255) return FS_ERR_INVALID_ARG;
    const TransposePlan pl = plan_transpose(M, K, nnz);
    if (scratch_bytes < pl.total_ints * sizeof(int)) return FS_ERR_BUFFER_TOO_SMALL;
    int *S = (int *)d_scratch;
    uint32_t *key[2] = {(uint32_t *)(S + pl.key0), (uint32_t *)(S + pl.key1)};
    int *hist = S + pl.hist, *tmp = S + pl.tmp, *first_of = S + pl.first_of;

    const uint32_t *src_key = (const uint32_t *)d_colidx;
    const int32_t *src_val = nullptr;
    const int P = pl.passes;
    for (int p = 0, shift = 0; p < P; shift += pl.bits[p++]) {
        const bool last = p == P - 1;
        uint32_t *dst_key = pl.rows && last ? (uint32_t *)d_colidx_t : key[p & 1];
        int32_t *dst_val = ((P - 1 - p) & 1) ? S + pl.val1 : d_perm;  // the last pass writes d_perm
        const SortRows rows{d_rowptr, M, pl.row_shift};
        int *starts = pl.rows && !last ? first_of : nullptr;
        auto pass = [&](auto bits_) -> fs_status {
            constexpr int BITS = decltype(bits_)::value;
            return pl.rows ? sort_pass<BITS, true>(src_key, src_val, nnz, 0, pl.bits[p], hist, tmp, dst_key, dst_val, st, rows, starts)
                           : sort_pass<BITS>(src_key, src_val, nnz, shift, pl.bits[p], hist, tmp, dst_key, dst_val, st);
        };
        const fs_status s = pl.bits[p] <= 8 ? pass(std::integral_constant<int, 8>{})
                            : pl.bits[p] == 9 ? pass(std::integral_constant<int, 9>{}) : pass(std::integral_constant<int, 10>{});
        if (s != FS_OK) return s;
        if (last && pl.rows) {
            const int low_bits = P == 2 ? pl.bits[0] : 0;
            k_rowptr_of_counts<<<(unsigned)((1 << low_bits) + 7) / 8 * 8, kCountsThreads, 0, st>>>(src_key, P == 2 ? first_of : nullptr, hist, (int)sort_groups(nnz),
                                                                              kSortWaves * sort_tile(nnz), low_bits, pl.bits[p], (int32_t)nnz, K, d_rowptr_t);
            FS_LAUNCH_CHECK();
            return FS_OK;
        }
        src_key = dst_key;
        src_val = dst_val;
    }
    // keys too wide to carry the rows along
    k_rowptr_of_sorted<<<grid_of(K + 1, 256), 256, 0, st>>>((const int32_t *)src_key, (int32_t)nnz, K, d_rowptr_t);
    FS_LAUNCH_CHECK();
    int32_t *row_of = (int32_t *)key[P & 1];  // the key buffer the last pass did not write
    int32_t *group_rows = hist;  // the digit counts are no longer needed; 256 a group + 1 >= nnz / 256 + 2 ints
    const int64_t n_groups = (nnz + kEntriesPerGroup - 1) / kEntriesPerGroup;
    k_group_rows<<<grid_of(n_groups + 1, 256), 256, 0, st>>>(d_rowptr, M, nnz, n_groups, group_rows);
    FS_LAUNCH_CHECK();
    k_row_of_entry<<<(unsigned)n_groups, kEntriesPerGroup, 0, st>>>(d_rowptr, nnz, group_rows, row_of);
    FS_LAUNCH_CHECK();
    k_gather_i32<<<grid_of(nnz, 256), 256, 0, st>>>(row_of, d_perm, nnz, d_colidx_t);
    FS_LAUNCH_CHECK();
    return FS_OK;
}

extern "C" fs_status fs_gather16(const void *d_src, const int32_t *d_idx, int64_t n, void *d_dst, void *stream)
{
    if (n < 0) return FS_ERR_INVALID_ARG;
    if (n == 0) return FS_OK;
    if (!d_src || !d_idx || !d_dst) return FS_ERR_INVALID_ARG;
    // One element a thread / sorted by band, a random permutation, us: 2 M elements 12.8 / 15, 3 M 23.7 / 19.8, 4.2 M 43 / 26.5,
    // 8 M 108 / 77, 20 M 334 / 294, 30 M 524 / 485.  A graph's permutation, in which neighbours come by again soon, gains less: R-MAT
    // of 512 k rows, 8 M 57 / 55; of 1 M rows, 31 M 298 / 360.
    // A look at the indices first costs nothing where all workgroups start at once on an idle memory (5.3 M random 38.2 / 38.1), and a
    // round trip through a busy one where they do not (10 M random 108 / 122); without it 8 M indices in order take 21 us for 18.
    const unsigned grid = grid_of(n, kBandThreads * kBandEach);
    const int shift = n <= (int64_t)kBands << 19 ? 19 : 20;  // bands of 1 or 2 MB
    const uint16_t *src = (const uint16_t *)d_src;
    uint16_t *dst = (uint16_t *)d_dst;
    if (n > ((int64_t)5 << 19) && n <= ((int64_t)3 << 21)) k_gather16_banded<true><<<grid, kBandThreads, 0, (hipStream_t)stream>>>(src, d_idx, n, shift, dst);
    else if (n > ((int64_t)5 << 19) && n <= ((int64_t)5 << 22)) k_gather16_banded<false><<<grid, kBandThreads, 0, (hipStream_t)stream>>>(src, d_idx, n, shift, dst);
    else k_gather16<<<grid_of(n, 256), 256, 0, (hipStream_t)stream>>>(src, d_idx, n, dst);
    FS_LAUNCH_CHECK();
    return FS_OK;
}
