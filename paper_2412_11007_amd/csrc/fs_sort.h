// One pass of a stable least-significant-digit radix sort on 8- or 9-bit digits of int32 keys, one wavefront per
// tile of 2048 entries, shared by the translation units that sort (the CSR transposition sorts entries by
// column; the conversion orders the work list).  Every translation unit gets its own copy.
//   hist     per tile, the number of entries per digit value
//   scan     (the caller's, fs_scan.h) exclusive prefix sum over (digit value, tile), digit-major: where
//            each tile's entries with a given digit start in the output
//   scatter  each wavefront walks its tile in order, 64 entries at a time; a lane's rank among the lanes
//            of the same digit comes from one wave-wide ballot per digit bit, so equal digits keep their input order;
//            four wavefronts (four consecutive tiles) share a workgroup and write their output together
// No atomics touch global memory and the result does not depend on scheduling.
#pragma once

#include <algorithm>

#include "fs_common.h"
#include "fs_scan.h"

namespace {

constexpr int kSortTile = 2048;       // entries per wavefront for large sorts
constexpr int kSortTileSmall = 256;   // ... and for sorts of a few thousand entries, where a wavefront's 32 sequential
                                      // rounds per 2048-entry tile would be the whole run time
// Digits of 8 bits, or of 9 where those make a pass fewer.  A wide pass costs more (twice the counts, one more ballot per
// round, 28 instead of 22 KB of LDS per workgroup), but two of them less than three narrow ones: transposition of 5.3 M
// entries with 18-bit columns 368 -> 350 us, 322 with the counting below.
constexpr int kDigitBits = 8, kWideDigitBits = 9;
constexpr int kDigits = 1 << kDigitBits, kWideDigits = 1 << kWideDigitBits;

constexpr int kScatterWaves = 4;
constexpr int kMaxRounds = kSortTile / 64;

// Four wavefronts count four consecutive tiles: their counts of one digit value are neighbours in hist, so they leave in
// 16-byte pieces, and a wavefront has eight loads in flight (5.3 M entries, 9 bits: 21.2 -> 10.4 us with a
// wavefront per workgroup, one load at a time and 4-byte stores before).
template <int BITS>
__global__ void __launch_bounds__(64 * kScatterWaves) k_digit_hist(const int32_t *__restrict__ keys, int64_t n, int shift, int64_t ntile,
                                                                   int *__restrict__ hist, int tile)
{
    constexpr int n_digits = 1 << BITS, kAhead = 8;
    __shared__ int h[kScatterWaves][n_digits];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kScatterWaves * n_digits; i += 64 * kScatterWaves) (&h[0][0])[i] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * kScatterWaves;
    const int64_t base = (t0 + w) * tile, end = std::min<int64_t>(base + tile, n);
    for (int64_t i0 = base + lane; i0 < end; i0 += 64 * kAhead) {
        int32_t key[kAhead];
#pragma unroll
        for (int r = 0; r < kAhead; r++) key[r] = keys[std::min<int64_t>(i0 + 64 * r, n - 1)];
#pragma unroll
        for (int r = 0; r < kAhead; r++)
            if (i0 + 64 * r < end) atomicAdd(&h[w][((uint32_t)key[r] >> shift) & (n_digits - 1)], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kScatterWaves * n_digits; i += 64 * kScatterWaves) {
        const int d = i / kScatterWaves, k = i % kScatterWaves;
        if (t0 + k < ntile) hist[(int64_t)d * ntile + t0 + k] = h[k][d];
    }
}

// Four wavefronts, four consecutive tiles.  In the output the entries of these tiles with a given digit are
// neighbours (the scan is digit-major, tile-minor), so the group's share of a digit is one run, four times
// as long as a tile's.  First every wavefront ranks its tile as above -- its keys are loaded up front, so the
// rounds wait for nothing but LDS -- and notes, for every output slot of the group, which entry goes there
// (a 16-bit index, 16 KB of LDS for the group); then the workgroup walks the output slots in order and
// fetches their entries again (they are still in cache), so that neighbouring lanes write neighbouring
// addresses: runs of ~128 bytes instead of scattered 4-byte pieces of ~32-byte runs.
// FIRST: the payload of entry i is i itself (its position in the source CSR order).
template <int BITS, bool FIRST>
__global__ void __launch_bounds__(64 * kScatterWaves)
k_digit_scatter(const int32_t *__restrict__ keys, const int32_t *__restrict__ vals, int64_t n, int shift, int64_t ntile,
                const int *__restrict__ start, int32_t *__restrict__ out_keys, int32_t *__restrict__ out_vals,
                int tile)
{
    constexpr int n_digits = 1 << BITS, kPer = n_digits / kScanThreads;  // kPer consecutive digit values per thread in the tables
    static_assert(64 * kScatterWaves == kScanThreads && kPer * kScanThreads == n_digits, "every digit value has a thread");
    __shared__ int cur[kScatterWaves][n_digits];  // where a tile's next entry with digit d goes in the output
    __shared__ int gbase[n_digits];               // where the group's entries with digit d start in the output ...
    __shared__ int lstart[n_digits];              // ... and among the group's own output slots
    __shared__ uint16_t source[kScatterWaves * kSortTile];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * kScatterWaves, t1 = std::min<int64_t>(t0 + kScatterWaves, ntile);
    {
        int count[kPer], sum = 0, tot;
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int d = threadIdx.x * kPer + i;
            const int g0 = start[(int64_t)d * ntile + t0];
            count[i] = start[(int64_t)d * ntile + t1] - g0;
            sum += count[i];
            gbase[d] = g0;
#pragma unroll
            for (int k = 0; k < kScatterWaves; k++) cur[k][d] = t0 + k < ntile ? start[(int64_t)d * ntile + t0 + k] : 0;
        }
        int ofs = block_exclusive_scan(sum, &tot);
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            lstart[threadIdx.x * kPer + i] = ofs;
            ofs += count[i];
        }
    }
    __syncthreads();
    const int64_t first = t0 * tile;  // the group's first entry
    const int64_t base = (t0 + w) * tile, end = std::min<int64_t>(base + tile, n);
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    int32_t key[kMaxRounds];
#pragma unroll
    for (int r = 0; r < kMaxRounds; r++) {
        const int64_t i = base + r * 64 + lane;
        key[r] = (r * 64 < tile && i < end) ? keys[i] : 0;
    }
#pragma unroll
    for (int r = 0; r < kMaxRounds; r++) {
        if (r * 64 >= tile || base + r * 64 >= end) break;  // the same for all lanes
        const int64_t i = base + r * 64 + lane;
        const bool valid = i < end;
        const int digit = ((uint32_t)key[r] >> shift) & (n_digits - 1);
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < BITS; b++) {
            const bool bit = (digit >> b) & 1;
            const uint64_t set = __ballot(valid && bit);
            same &= bit ? set : ~set;
        }
        const int rank = __popcll(same & below), cnt = __popcll(same);
        int pos = 0;
        if (valid) {
            pos = cur[w][digit];
            source[pos + rank - gbase[digit] + lstart[digit]] = (uint16_t)(i - first);
        }
        __builtin_amdgcn_wave_barrier();  // the wavefront's reads above stay before its update below
        if (valid && rank == cnt - 1) cur[w][digit] = pos + cnt;
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    const int total = (int)(std::min<int64_t>(t1 * tile, n) - first);
#pragma unroll 4
    for (int s = threadIdx.x; s < total; s += 64 * kScatterWaves) {
        const int64_t i = first + source[s];
        const int32_t k = keys[i];
        const int32_t v = FIRST ? (int32_t)i : vals[i];
        const int digit = ((uint32_t)k >> shift) & (n_digits - 1);
        const int pos = gbase[digit] + (s - lstart[digit]);
        out_keys[pos] = k;
        out_vals[pos] = v;
    }
}

// One pass: keys (and payload; null: an entry's position) to out_keys and out_vals.  hist: 2^BITS * ntile + 1 ints,
// tmp: what a scan of them takes.
template <int BITS>
fs_status sort_pass(const int32_t *keys, const int32_t *vals, int64_t n, int shift, int tile, int *hist, int *tmp, int32_t *out_keys,
                    int32_t *out_vals, hipStream_t st)
{
    const int64_t ntile = (n + tile - 1) / tile;
    const dim3 grid((unsigned)((ntile + kScatterWaves - 1) / kScatterWaves)), block(64 * kScatterWaves);
    k_digit_hist<BITS><<<grid, block, 0, st>>>(keys, n, shift, ntile, hist, tile);
    FS_LAUNCH_CHECK();
    const fs_status s = scan_exclusive(hist, ntile << BITS, tmp, st);
    if (s != FS_OK) return s;
    if (!vals) k_digit_scatter<BITS, true><<<grid, block, 0, st>>>(keys, nullptr, n, shift, ntile, hist, out_keys, out_vals, tile);
    else k_digit_scatter<BITS, false><<<grid, block, 0, st>>>(keys, vals, n, shift, ntile, hist, out_keys, out_vals, tile);
    FS_LAUNCH_CHECK();
    return FS_OK;
}

}  // namespace
