// One pass of a stable least-significant-digit radix sort of (key, payload) pairs of 32 bits each, on digits of up to 8,
// 9 or 10 bits, shared by the translation units that sort (the CSR transposition sorts entries by column; the conversion
// orders the work list).  Every translation unit gets its own copy.
//   hist     per group of eight tiles, the number of entries per digit value
//   scan     (fs_scan.h) exclusive prefix sum over (digit value, group), digit-major: where each group's entries with a
//            given digit start in the output
//   scatter  one workgroup per group, one wavefront per tile: a wavefront ranks its tile 64 entries at a time (a lane's
//            rank among the lanes of the same digit comes from one wave-wide ballot per digit bit, so equal digits keep
//            their input order), then the group's keys and its payloads pass through LDS in output order
// No atomics touch global memory and the result does not depend on scheduling.
//
// What bounds a pass is the memory side of the scatter, so its stores are made as long as they can be: neighbouring lanes
// write neighbouring addresses (a digit's run of a group: 16 entries of 4 bytes on average at 9 bits), and consecutive groups,
// whose runs of one digit follow each other in the output, run on one XCD, where its L2 puts them together to whole lines.
// Fetching the entries again in output order instead of passing them through LDS cost two scattered lines an entry:
// 5.3 M entries, 9-bit digits, 48 us (first pass) and 70 us, now 35 (the rows looked up on the way) and 31: 84 MB, 2.7 TB/s.
#pragma once

#include <algorithm>

#include "fs_common.h"
#include "fs_scan.h"
#include "fs_tile.h"  // FS_WAVE_SYNC

namespace {

constexpr int kSortWaves = 8;                   // tiles per group
constexpr int kSortThreads = 64 * kSortWaves;
constexpr int kSortTile = 1024;                 // most entries per tile
constexpr int kSortRounds = kSortTile / 64;
constexpr int kMaxDigitBits = 10;
static_assert(kSortWaves * kSortTile <= 1 << 13, "a place in a group has 13 bits");

// Entries per tile: as many as make 256 groups (a workgroup per CU), within 128 (fewer make the counts outgrow the
// entries) and kSortTile.  (A work list of 98 k items, 8-bit digits: 21 us a scatter on twelve groups, 7 on 96.)
inline int sort_tile(int64_t n) { return (int)std::min<int64_t>(std::max<int64_t>((n / (256 * kSortWaves) + 64) / 64 * 64, 128), kSortTile); }
inline int64_t sort_groups(int64_t n) { return (n + kSortWaves * sort_tile(n) - 1) / (kSortWaves * sort_tile(n)); }
// ... and the most groups of any number of entries up to n
inline int64_t sort_groups_bound(int64_t n) { return std::max<int64_t>(std::min<int64_t>(n / (kSortWaves * 128) + 1, 257), n / (kSortWaves * kSortTile) + 1); }

// Workgroup b's group: XCD b % 8 takes an eighth of the groups, one after the other.
__device__ __forceinline__ int sort_group(int ngroup)
{
    const int per = (ngroup + 7) / 8;
    return (blockIdx.x & 7) * per + (blockIdx.x >> 3);
}

// digit = key >> shift & mask
template <int BITS>
__global__ void __launch_bounds__(kSortThreads) k_digit_hist(const uint32_t *__restrict__ keys, int64_t n, int shift, uint32_t mask, int ngroup,
                                                             int *__restrict__ hist, int tile)
{
    constexpr int n_digits = 1 << BITS, kCopies = 4, kAhead = 8;
    __shared__ int h[kCopies][n_digits];
    const int grp = sort_group(ngroup);
    if (grp >= ngroup) return;
    for (int i = threadIdx.x; i < kCopies * n_digits; i += kSortThreads) (&h[0][0])[i] = 0;
    __syncthreads();
    int *mine = h[(threadIdx.x >> 6) % kCopies];
    const int64_t first = (int64_t)grp * kSortWaves * tile, end = std::min<int64_t>(first + kSortWaves * tile, n);
    for (int64_t i0 = first + threadIdx.x; i0 < end; i0 += kSortThreads * kAhead) {
        uint32_t key[kAhead];
#pragma unroll
        for (int r = 0; r < kAhead; r++) key[r] = keys[std::min<int64_t>(i0 + kSortThreads * r, n - 1)];
#pragma unroll
        for (int r = 0; r < kAhead; r++)
            if (i0 + kSortThreads * r < end) atomicAdd(&mine[key[r] >> shift & mask], 1);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < n_digits; d += kSortThreads) {
        int c = 0;
#pragma unroll
        for (int k = 0; k < kCopies; k++) c += h[k][d];
        hist[(int64_t)d * ngroup + grp] = c;
    }
}

// The rows of a sort that carries them along (the transposition): in the first pass the key of entry i is its column, and
// what goes on is the column without this pass's digit and, from bit `shift` on, the row that stores entry i; later passes
// drop their digits as well, so that the last one leaves the row alone.  The digits are then always the lowest bits.
struct SortRows {
    const int32_t *rowptr;  // null: keys are sorted as they are, and stay whole
    int64_t M;
    int shift;
};

// The last rows of [0, M) whose pointer is at most p0 and p1, by the whole wavefront: 64 probes a step.  Stays inside
// [0, M) whatever rowptr holds.
__device__ __forceinline__ void wave_rows_of(const int32_t *__restrict__ rowptr, int64_t M, int64_t p0, int64_t p1, int64_t &r0, int64_t &r1)
{
    const int lane = threadIdx.x & 63;
    int64_t lo[2] = {0, 0}, len = M;
    while (len > 1) {
        const int64_t step = (len + 63) / 64;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int64_t at = lo[k] + lane * step;
            const int32_t v = rowptr[std::min<int64_t>(at, M - 1)];
            const uint64_t upto = __ballot(lane * step < len && at < M && v <= (k ? p1 : p0));
            lo[k] += (int64_t)(upto ? 63 - __builtin_clzll(upto) : 0) * step;
        }
        len = step;
    }
    r0 = lo[0];
    r1 = lo[1];
}

// A loop whose index is a constant from the start, so that arrays of a lane's entries stay in registers of their own
// (unrolled late, they are a tuple that every branch copies).
#define FS_ROUND(r) fs_for_each_index([&](auto r##_) { constexpr int r = decltype(r##_)::value;
#define FS_ROUND_END }, std::make_integer_sequence<int, kSortRounds>{})

// FIRST: the payload of entry i is i itself.  ROWS: see SortRows; `first_of` (optional) receives where each digit's
// entries start in the output.
template <int BITS, bool FIRST, bool ROWS>
__global__ void __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(6)))
k_digit_scatter(const uint32_t *__restrict__ keys, const int32_t *__restrict__ vals, int64_t n, int shift, int bits, int ngroup,
                const int *__restrict__ start, uint32_t *__restrict__ out_keys, int32_t *__restrict__ out_vals, int tile, SortRows rows,
                int *__restrict__ first_of)
{
    constexpr int n_digits = 1 << BITS, kPer = (n_digits + kSortThreads - 1) / kSortThreads;  // consecutive digit values of a thread
    __shared__ uint32_t stage[kSortWaves * kSortTile];
    __shared__ uint16_t cur[kSortWaves][n_digits];  // a tile's entries so far per digit; then where they start among the group's
    __shared__ int delta[n_digits];                 // place in the output minus place in the group
    __shared__ uint32_t opens[ROWS && FIRST ? kSortWaves : 1][2 * kSortRounds];  // a bit per entry that opens a row
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int grp = sort_group(ngroup);
    if (grp >= ngroup) return;  // the same for the workgroup
    const uint32_t mask = (1u << bits) - 1;
    const int64_t first = (int64_t)grp * kSortWaves * tile;  // the group's first entry
    // from here on entries are counted from the group's first
    const int left = (int)std::min<int64_t>(n - first, kSortWaves * tile), base = w * tile, end = std::min(base + tile, left);
    keys += first;
    if constexpr (!FIRST) vals += first;
    uint32_t key[kSortRounds];
    int32_t val[FIRST ? 1 : kSortRounds];
    uint32_t pos[kSortRounds];  // place in the tile's share of the digit, later in the group | digit << 16
    FS_ROUND(r)
        const int i = base + r * 64 + lane;
        key[r] = keys[(uint32_t)std::min(i, left - 1)];
        if constexpr (!FIRST) val[r] = vals[(uint32_t)std::min(i, left - 1)];
    FS_ROUND_END;
    int at_start[kPer];
#pragma unroll
    for (int i = 0; i < kPer; i++) {
        const int d = threadIdx.x * kPer + i;
        at_start[i] = d < n_digits ? start[(int64_t)d * ngroup + grp] : 0;
        if (first_of && grp == 0 && d < n_digits) first_of[d] = at_start[i];
    }
    for (int d = lane; d < n_digits; d += 64) cur[w][d] = 0;
    __builtin_amdgcn_wave_barrier();
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    FS_ROUND(r)
        pos[r] = 0;
        asm volatile("" : "+v"(key[r]) : : "memory");  // one round after the other: run ahead, their ballots would fill the registers
        if (base + r * 64 < end) {  // the same for all lanes
            const bool valid = base + r * 64 + lane < end;
            const uint32_t digit = key[r] >> shift & mask;
            uint64_t same = __ballot(valid);
#pragma unroll
            for (int b = 0; b < BITS; b++) {
                const bool bit = (digit >> b) & 1;
                const uint64_t set = __ballot(valid && bit);
                same &= bit ? set : ~set;
            }
            const int rank = __popcll(same & below), cnt = __popcll(same);
            const int at = cur[w][digit];
            pos[r] = (uint32_t)(at + rank) | digit << 16;
            __builtin_amdgcn_wave_barrier();  // the wavefront's reads above stay before its update below
            if (valid && rank == cnt - 1) cur[w][digit] = (uint16_t)(at + cnt);
            __builtin_amdgcn_wave_barrier();
        }
    FS_ROUND_END;
    if constexpr (ROWS && FIRST) {
        // Rows of the tile's entries: a bit per entry that opens a row and a list of those rows (where the group's entries
        // will be staged); an entry's row is the one on the list at the number of set bits up to the entry.
        uint32_t *list = stage + w * kSortTile;
        int64_t r0 = 0, r1 = 0;
        if (base < end) wave_rows_of(rows.rowptr, rows.M, first + base, first + end - 1, r0, r1);
        if (r1 - r0 <= 8 * kSortTile) {
            if (lane < 2 * kSortRounds) opens[w][lane] = 0;
            if (lane == 0) list[0] = (uint32_t)r0;
            FS_WAVE_SYNC();
            int listed = 1;
            for (int64_t ra = r0 + 1; ra <= r1; ra += 64) {
                const int64_t row = ra + lane;
                const int64_t at = rows.rowptr[std::min(row, r1)] - first - base;
                const bool some = row <= r1 && rows.rowptr[std::min(row, r1) + 1] - first - base > at && at > 0 && at < tile;
                const uint64_t set = __ballot(some);
                const int k = listed + __popcll(set & below);
                if (some && k < kSortTile) {  // (always, for pointers that do not descend)
                    list[k] = (uint32_t)row;
                    atomicOr(&opens[w][at >> 5], 1u << (at & 31));
                }
                listed += __popcll(set);
            }
            FS_WAVE_SYNC();
            int before = 0;
            FS_ROUND(r)
                if (base + r * 64 < end) {
                    const uint64_t set = opens[w][2 * r] | (uint64_t)opens[w][2 * r + 1] << 32;
                    key[r] = key[r] >> bits | list[before + __popcll(set & (below << 1 | 1))] << rows.shift;
                    before += __popcll(set);
                }
            FS_ROUND_END;
        } else {  // mostly empty rows: search among them
            for (int i = base + lane; i < end; i += 64) {
                int64_t lo = r0, hi = r1 + 1;  // the last row that starts at the entry or before
                while (hi - lo > 1) {
                    const int64_t mid = lo + ((hi - lo) >> 1);
                    if (rows.rowptr[mid] <= first + i) lo = mid; else hi = mid;
                }
                list[i - base] = (uint32_t)lo;
            }
            FS_WAVE_SYNC();
            FS_ROUND(r)
                if (base + r * 64 < end) key[r] = key[r] >> bits | list[r * 64 + lane] << rows.shift;
            FS_ROUND_END;
        }
    }
    __syncthreads();
    {
        int count[kPer], sum = 0, tot;
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int d = threadIdx.x * kPer + i;
            count[i] = 0;
            if (d < n_digits) {
#pragma unroll
                for (int k = 0; k < kSortWaves; k++) count[i] += cur[k][d];
            }
            sum += count[i];
        }
        int ofs = block_exclusive_scan<kSortThreads>(sum, &tot);
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int d = threadIdx.x * kPer + i;
            if (d < n_digits) {
                delta[d] = at_start[i] - ofs;
#pragma unroll
                for (int k = 0; k < kSortWaves; k++) {
                    const int c = cur[k][d];
                    cur[k][d] = (uint16_t)ofs;
                    ofs += c;
                }
            }
        }
    }
    __syncthreads();
    // The word that tells an output place's digit goes through LDS first: the key, or, where the key has lost the digit or is
    // not needed for it, the payload beside the digit.
    FS_ROUND(r)
        if (base + r * 64 + lane < end) {
            const uint32_t digit = pos[r] >> 16;
            pos[r] = cur[w][digit] + (pos[r] & 0xFFFF);
            stage[pos[r]] = FIRST ? (uint32_t)(base + r * 64 + lane) | digit << 13 : key[r];
        }
    FS_ROUND_END;
    __syncthreads();
    uint32_t to[kSortRounds];
    FS_ROUND(k)
        const int s = k * kSortThreads + threadIdx.x;
        to[k] = 0;
        if (s < left) {
            const uint32_t x = stage[s];
            to[k] = s + delta[FIRST ? x >> 13 : (x >> shift & mask)];
            if constexpr (FIRST) out_vals[to[k]] = (int32_t)(first + (x & 8191));
            else out_keys[to[k]] = ROWS ? x >> bits : x;
        }
    FS_ROUND_END;
    __syncthreads();
    FS_ROUND(r)
        if (base + r * 64 + lane < end) stage[pos[r]] = FIRST ? key[r] : (uint32_t)val[FIRST ? 0 : r];
    FS_ROUND_END;
    __syncthreads();
    FS_ROUND(k)
        const int s = k * kSortThreads + threadIdx.x;
        if (s < left) {
            if constexpr (FIRST) out_keys[to[k]] = stage[s];
            else out_vals[to[k]] = (int32_t)stage[s];
        }
    FS_ROUND_END;
}
#undef FS_ROUND
#undef FS_ROUND_END

// One pass on the `bits` bits from `shift` on: keys (and payload; null: an entry's position) to out_keys and out_vals.
// hist: 2^BITS * sort_groups(n) + 1 ints, tmp: what a scan of them takes.
template <int BITS, bool ROWS = false>
fs_status sort_pass(const uint32_t *keys, const int32_t *vals, int64_t n, int shift, int bits, int *hist, int *tmp, uint32_t *out_keys,
                    int32_t *out_vals, hipStream_t st, SortRows rows = SortRows{}, int *first_of = nullptr)
{
    const int tile = sort_tile(n), ngroup = (int)sort_groups(n);
    const unsigned grid = (unsigned)((ngroup + 7) / 8 * 8);
    k_digit_hist<BITS><<<grid, kSortThreads, 0, st>>>(keys, n, shift, (1u << bits) - 1, ngroup, hist, tile);
    FS_LAUNCH_CHECK();
    const fs_status s = scan_exclusive(hist, (int64_t)ngroup << BITS, tmp, st);
    if (s != FS_OK) return s;
    if (!vals) k_digit_scatter<BITS, true, ROWS><<<grid, kSortThreads, 0, st>>>(keys, nullptr, n, shift, bits, ngroup, hist, out_keys, out_vals, tile, rows, first_of);
    else k_digit_scatter<BITS, false, ROWS><<<grid, kSortThreads, 0, st>>>(keys, vals, n, shift, bits, ngroup, hist, out_keys, out_vals, tile, rows, first_of);
    FS_LAUNCH_CHECK();
    return FS_OK;
}

}  // namespace
