// The conversion's units of work and the two kernels that walk them: one ranks every stored entry among its
// window's nonzero vectors, the other writes the format's arrays from those ranks.
//
// A unit is at most kUnitEntries stored entries, handled by one wavefront in LDS: a few consecutive windows, one
// window, or -- of a hub window with more entries than that -- a range of columns.  What bounds the conversion
// otherwise is searching: with one thread per entry and a binary search in each of the window's other rows, every
// probe is a cache line (31.4 M entries in eight-row windows: 1.7 ms in two such kernels).  In LDS a unit's distinct columns are
// counted in order by the bits of a trie (k_unit_rank).  Those entries (R-MAT of 1 M rows): the whole conversion 2.70 -> 0.77 ms, of which
// ranking takes 119 us and placing 315 us (1.2 GB, most of it written, 260 us).
#pragma once

#include <algorithm>

#include "fs_common.h"
#include "fs_scan.h"
#include "fs_tile.h"  // FS_WAVE_SYNC: a barrier would also wait for every store under way

namespace {

// Waits for every load under way.  The kernels below issue all of a unit's loads under uniform branches and use them
// under others; without one place at which all have arrived, the compiler waits for everything in flight -- the stores
// included -- wherever it cannot tell.
#define FS_WAIT_LOADS() __builtin_amdgcn_s_waitcnt(0x0F70)  /* vmcnt(0), nothing else */

// A loop over the up to NCH entries of a lane whose index is a constant from the start, so that arrays of them stay in
// registers of their own (unrolled late, the compiler had made one of them a tuple that every branch copied).
#define FS_EACH(h) fs_for_each_index([&](auto h##_) { constexpr int h = decltype(h##_)::value;
#define FS_EACH_END }, std::make_integer_sequence<int, NCH>{})

constexpr int kUnitEntries = 512;   // 9 bits of a rank
constexpr int kUnitRows = 64;       // rows of a unit, one per lane: 6 bits
constexpr int kMaxUnitWindows = 16;

struct CsrView {
    const int32_t *rowptr;
    const int32_t *colidx;
    int64_t M;
    int32_t nnz;
};

// Row bounds clamped into [0, nnz] so that a malformed rowptr can never cause an out-of-range read.
__device__ __forceinline__ void row_range(const CsrView &a, int64_t i, int32_t &lo, int32_t &hi)
{
    lo = min(max(a.rowptr[i], 0), a.nnz);
    hi = min(max(a.rowptr[i + 1], lo), a.nnz);
}

// How windows become units.  Windows are taken in groups of `group`, as many as have at most kUnitRows rows; a group of up to `fill`
// entries is a unit, else its halves are looked at, and so on: a unit is the largest aligned run of 2^k windows that fits.  (With one
// size of run for the whole matrix, the short windows beside the hubs of a power-law graph were units of their own: R-MAT
// of 1 M rows, 32 a row, 202 k units of 156 entries, now 100 k of 314: ranking 297 -> 239 us, placing 419 -> 320.)  `fill` is kUnitEntries, but
// less on matrices that would not make four units a CU: there a wavefront's own chain is the time (4096 rows, 16 a row, with
// full units 132 us, filled to 128 entries 123).  A window with more than kUnitEntries entries is cut by columns:
// every `stride`-th entry of a row is a sample, a sample's rank counts the samples of all rows with a smaller
// (column, row), and the columns of the samples with ranks `per`, 2 per, ... start new pieces.  A piece then
// spans at most per + V - 1 samples, a row with q of them at most (q + 1) * stride - 1 entries of it: in all fewer than
// (per + 2 V) * stride <= kUnitEntries.  (`per` stays a sixth below what that allows, so that pieces cut by a guess
// fit as well, see k_pieces.)
struct UnitPlan {
    int V, lv;     // rows per window, and log2 of the next power of two
    int group;     // windows per group, a power of two
    int fill;      // most entries of a unit of several windows
    int stride, per;
};
inline UnitPlan unit_plan(int64_t nnz, int V)
{
    UnitPlan p;
    p.V = V;
    p.lv = 0;
    while ((1 << p.lv) < V) p.lv++;
    p.group = std::min(kMaxUnitWindows, kUnitRows >> p.lv);
    p.fill = (int)std::min<int64_t>(std::max<int64_t>(nnz / 1024, 128), kUnitEntries);
    p.stride = 4;
    p.per = (kUnitEntries / p.stride - 2 * V) * 5 / 6;
    return p;
}
// At most this many units, for every V (per * stride >= 212): what the scratch buffer has room for.
inline int64_t units_bound(int64_t W, int64_t nnz) { return W + nnz / 208 + 2; }
// ... and for a plan: a unit per group; of the at most nnz / (fill + 1) groups that do not fit one, at most a unit per window;
// of a hub window one more per (per * stride) entries.  (Launched for the bound above, a matrix with fewer entries than
// rows ran mostly empty workgroups: 16 M rows, 1 M entries, four-row windows 3.49 -> 1.09 ms.)
inline int64_t units_bound(const UnitPlan &p, int64_t W, int64_t nnz)
{
    const int64_t groups = (W + p.group - 1) / p.group;
    return std::min(groups + (p.group - 1) * (nnz / (p.fill + 1)), W) + nnz / (p.per * p.stride) + 2;
}
// Workgroups per launch: a launch has fewer than 2^32 threads, so a larger number takes several.
template <typename Launch>
fs_status launch_units(int64_t n, Launch launch, int waves = 1)
{
    const int64_t most = ((int64_t)1 << 24) / waves;
    for (int64_t first = 0; first < n; first += most) {
        launch((int)first, (unsigned)std::min(n - first, most));
        FS_LAUNCH_CHECK();
    }
    return FS_OK;
}

// Units that begin with a window, one window per lane (groups are aligned runs of lanes).  run: windows of the unit, 0 if none
// begins here; n: 1, or the pieces of a hub window.
struct WindowUnits {
    int run, n;
};
// first, end: the window's entries (of windows past the last: none, at the matrix' end); samples(): of a hub window, what its rows hold
template <typename Samples>
__device__ __forceinline__ WindowUnits window_units(const UnitPlan &p, int k, int32_t first, int32_t end, bool exists, Samples samples)
{
    WindowUnits x{0, 0};
    const int lane = threadIdx.x & 63;
    bool hub = true;
    for (int run = p.group; run >= 1; run >>= 1) {  // the largest aligned run around the window that fits
        const int from = lane & -run;
        const int e = __shfl(end, from + run - 1, 64) - __shfl(first, from, 64);
        if (hub && e <= (run > 1 ? p.fill : kUnitEntries)) {
            hub = false;
            if (exists && (k & (run - 1)) == 0) x = WindowUnits{run, 1};
        }
    }
    if (exists && hub) x = WindowUnits{1, (int)max((samples() + p.per - 1) / p.per, (int64_t)1)};
    return x;
}

// How many units the windows of every workgroup of k_units_fill become, and a check of the row pointers.  A workgroup takes `tiles` tiles of
// kCountGroups groups; the row pointers of a tile pass through LDS, so that they are read side by side (16 M rows: 155 us read by each
// thread for itself, now 36).
constexpr int kCountThreads = 256, kCountGroups = 32;
__global__ void __launch_bounds__(kCountThreads) k_units_count(CsrView a, UnitPlan p, int64_t W, int tiles, int *__restrict__ made, int *__restrict__ err)
{
    constexpr int kMost = kCountGroups * kUnitRows + 1, kAhead = 8;
    __shared__ int32_t rp[kMost + kMost / 32 + 1];
    auto at = [](int i) -> int { return i + (i >> 5); };  // windows are often a power of two apart: spread them over the banks
    bool bad = false;
    int n = 0;
    for (int tile = 0; tile < tiles; tile++) {
        const int64_t w0 = ((int64_t)blockIdx.x * tiles + tile) * kCountGroups * p.group, row0 = w0 * p.V;
        if (w0 >= W && w0 > 0) break;
        const int here = (int)min((int64_t)kCountGroups * p.group * p.V, a.M - row0);
        if (tile > 0) __syncthreads();
        for (int i0 = threadIdx.x; i0 <= here; i0 += kAhead * kCountThreads) {
            int32_t v[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; k++) v[k] = a.rowptr[row0 + min(i0 + k * kCountThreads, here)];
#pragma unroll
            for (int k = 0; k < kAhead; k++) rp[at(min(i0 + k * kCountThreads, here))] = v[k];
        }
        __syncthreads();
        if (threadIdx.x == 0) bad |= (w0 == 0 && rp[0] != 0) || (row0 + here == a.M && rp[at(here)] != a.nnz);
        for (int i = threadIdx.x; i < kCountGroups * p.group; i += kCountThreads) {  // (the same for the lanes of a wavefront)
            const int lo = min(i * p.V, here), hi = min(lo + p.V, here);
            for (int r = lo; r < hi; r++) bad |= rp[at(r + 1)] < rp[at(r)];
            n += window_units(p, i & (p.group - 1), rp[at(lo)], rp[at(hi)], w0 + i < W, [&]() -> int64_t {
                int64_t samples = 0;
                for (int r = lo; r < hi; r++) samples += max(rp[at(r + 1)] - rp[at(r)], 0) / p.stride;
                return samples;
            }).n;  // (of malformed row pointers any number: nothing is made of it)
        }
    }
    if (bad) atomicOr(err, 1);
    int total[1] = {n};
    block_sum<kCountThreads>(total);
    if (threadIdx.x == 0) made[blockIdx.x] = total[0];
}

// One window per thread again: the records {first window, windows, piece, pieces of the window} of the units that begin with it, in
// the order of the windows.  made = the workgroups' counts, of which each adds up those before its own: at most kScanDirect.  The many
// records of a hub window are written by the whole wavefront (a row of 5 M entries, 16 k records: 346 us by one thread, now 10).
__global__ void __launch_bounds__(kCountThreads) k_units_fill(CsrView a, UnitPlan p, int64_t W, int tiles, const int *__restrict__ made, int4 *__restrict__ units,
                                                              int *__restrict__ n_units, int *__restrict__ redo, const int *__restrict__ err)
{
    if (*err & 1) return;
    const int lane = threadIdx.x & 63, per_tile = kCountGroups * p.group;
    int before[1] = {0};
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += kCountThreads) before[0] += made[k];
    block_sum<kCountThreads>(before);
    int ahead = before[0];
    for (int64_t i0 = 0; i0 < (int64_t)tiles * per_tile; i0 += kCountThreads) {
        const int64_t w = (int64_t)blockIdx.x * tiles * per_tile + i0 + threadIdx.x;
        const bool mine = i0 + threadIdx.x < (int64_t)tiles * per_tile && w < W;  // (few windows a group: a tile has fewer than threads)
        const int64_t lo = min(w * p.V, a.M), hi = min(lo + p.V, a.M);
        const WindowUnits x = window_units(p, lane & (p.group - 1), a.rowptr[lo], a.rowptr[hi], mine, [&]() -> int64_t {
            int64_t n = 0;
            for (int64_t r = lo; r < hi; r++) n += (a.rowptr[r + 1] - a.rowptr[r]) / p.stride;
            return n;
        });
        int here;
        const int u = ahead + block_exclusive_scan<kCountThreads>(x.n, &here);
        ahead += here;
        if (x.n == 1) units[u] = make_int4((int)w, (int)min((int64_t)x.run, W - w), 0, 1);
        if (x.n > 1) redo[w] = 0;
        constexpr int kFew = 16;
        if (x.n > 1 && x.n <= kFew)
            for (int q = 0; q < x.n; q++) units[u + q] = make_int4((int)w, 1, q, x.n);
        for (uint64_t todo = __ballot(x.n > kFew); todo; todo &= todo - 1) {
            const int l = __builtin_ctzll(todo), first = __shfl(u, l, 64), many = __shfl(x.n, l, 64), of = __shfl((int)w, l, 64);
            for (int q = lane; q < many; q += 64) units[first + q] = make_int4(of, 1, q, many);
        }
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *n_units = ahead;
}

// First position in [lo, hi) whose column is >= c.
__device__ __forceinline__ int32_t first_at_least(const int32_t *__restrict__ colidx, int32_t lo, int32_t hi, int32_t c)
{
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (colidx[mid] < c) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Where the pieces of hub windows start: start[u * V + r] = the first entry of row r that belongs to piece u or a later
// one.  Piece k should start where k / pieces of the window's entries lie before; that column is looked for among
// those of the window's longest row, by interpolation between the two nearest ones known (a guess from the longest
// row alone is off by a factor where the hot columns saturate all rows).  A search in a row is a probe a lane, and the probes are the
// time; so a step ends the search as soon as a piece that is off at both ends still fits a unit, and later steps look
// near by first (R-MAT of 1 M rows 68 -> 61 us, of 65 k rows 13 -> 10).  A few steps are enough for a graph; a window
// one of whose pieces came out too large for a unit is noted in redo[] for k_pieces_exact.  64 / ROWS pieces per
// wavefront, one row per lane; the last one of a wavefront is only there for the size of the one before.
template <int ROWS>  // a power of two, at least V
__global__ void __launch_bounds__(64) k_pieces(int block0, CsrView a, UnitPlan p, const int4 *__restrict__ units, const int *__restrict__ n_units,
                                               int32_t *__restrict__ start, int *__restrict__ redo, const int *__restrict__ err)
{
    constexpr int PER = 64 / ROWS;
    const int close = (kUnitEntries - p.per * p.stride) / 2;  // near enough: a piece too long at both ends still fits
    const int lane = threadIdx.x, k = lane / ROWS, r = lane % ROWS;
    const int u0 = (block0 + blockIdx.x) * (PER - 1), u = u0 + k, n = *n_units;
    if (u0 >= n || (*err & 1)) return;
    const int4 un = units[min(u, n - 1)];
    const bool hub = u < n && un.w > 1;
    if (!__any(hub)) return;
    const int64_t row = (int64_t)un.x * p.V + r;
    int32_t lo = 0, hi = 0;
    if (hub && r < p.V && row < a.M) row_range(a, row, lo, hi);
    auto over_rows = [](int v) -> int {
#pragma unroll
        for (int h = 1; h < ROWS; h <<= 1) v += __shfl_xor(v, h, 64);
        return v;
    };
    uint64_t best = ((uint64_t)(uint32_t)(hi - lo) << 32) | (uint32_t)lo;  // the longest row's length and place
#pragma unroll
    for (int h = 1; h < ROWS; h <<= 1) {
        const uint64_t other = __shfl_xor(best, h, 64);
        best = other > best ? other : best;
    }
    const int32_t long_lo = (int32_t)(uint32_t)best, long_len = (int32_t)(best >> 32);
    const int all = over_rows(hi - lo);
    const int want = hub ? (int)((int64_t)all * un.z / un.w) : 0;
    // between which places of the longest row the column lies, and what of this row and of all lies before them
    int i_lo = 0, i_hi = long_len, f_lo = 0, f_hi = all;
    int32_t at_lo = lo, at_hi = hi, at = lo;
    int off = 0;  // entries by which the last column was off
    bool done = !hub || un.z == 0;
    for (int step = 0; step < 6 && !__all(done); step++) {
        int i = i_lo + (int)((int64_t)(want - f_lo) * (i_hi - i_lo) / max(f_hi - f_lo, 1));
        if (step == 3) i = (i_lo + i_hi) >> 1;
        i = min(max(i, i_lo), long_len - 1);
        if (!done) {
            const int32_t c = a.colidx[long_lo + i];
            int32_t from = at_lo, to = at_hi;
            if (off != 0) {  // the row's share of what is missing, twice over, is mostly more than enough
                const int reach = 2 * (int)((int64_t)abs(off) * (hi - lo) / max(all, 1)) + 8;
                const int32_t q = off < 0 ? from + reach : to - 1 - reach;
                if (q >= from && q < to) {
                    if (a.colidx[q] < c) from = q + 1; else to = q;
                }
            }
            at = first_at_least(a.colidx, from, to, c);
        }
        const int f = over_rows(at - lo);
        if (!done) {
            off = f - want;
            if (abs(off) <= close || i_hi - i_lo <= 1) done = true;
            if (f < want) { i_lo = i + 1; f_lo = f; at_lo = at; }
            else { i_hi = i; f_hi = f; at_hi = at; }
            if (i_lo >= i_hi) done = true;
        }
    }
    if (hub && r < p.V) start[(int64_t)u * p.V + r] = at;
    // entries of piece k: up to where the next one starts, or the rows' ends
    const int32_t next = __shfl(at, (lane + ROWS) & 63, 64);
    const int size = over_rows(hub && k < PER - 1 ? (un.z + 1 < un.w ? next : hi) - at : 0);
    const bool behind = hub && k < PER - 1 && un.z + 1 < un.w && next < at;  // pieces out of order
    if ((size > kUnitEntries || behind) && hub) redo[un.x] = 1;
}

// The same without a guess, for the windows in redo[].  The wavefront of piece k ranks the samples k * per .. of its window, numbered row after row; the sample
// whose rank is q * per starts piece q with its column.  (Ranks are distinct, so every piece of a valid matrix is
// written once.)  Counting a row's samples below the column leaves `stride` entries to look at for the row's start.
// The rows are searched eight at a time: one memory round trip per halving, not eight.
constexpr int kExactPerWave = 4;  // units a wavefront looks at
template <int ROWS>  // at least V, a multiple of eight
__global__ void __launch_bounds__(64) k_pieces_exact(int block0, CsrView a, UnitPlan p, const int4 *__restrict__ units, const int *__restrict__ n_units,
                                               int32_t *__restrict__ start, const int *__restrict__ redo, const int *__restrict__ err)
{
    constexpr int G = 8;
    const int lane = threadIdx.x, n = *n_units;
    if (*err & 1) return;
    const int u0 = (block0 + blockIdx.x) * kExactPerWave, my_u = u0 + lane;  // most have nothing to do
    const int4 my_un = units[min(my_u, n - 1)];
    uint64_t todo = __ballot(lane < kExactPerWave && my_u < n && my_un.w > 1 && redo[my_un.x]);
    for (; todo; todo &= todo - 1) {
        const int k = __builtin_ctzll(todo), u = u0 + k;
        const int4 un = make_int4(__shfl(my_un.x, k, 64), 1, __shfl(my_un.z, k, 64), __shfl(my_un.w, k, 64));
        const int64_t row0 = (int64_t)un.x * p.V;
        int32_t lo = 0, hi = 0;
        if (lane < p.V && row0 + lane < a.M) row_range(a, row0 + lane, lo, hi);
        if (un.z == 0 && lane < p.V) start[(int64_t)u * p.V + lane] = lo;
        const int mine = (hi - lo) / p.stride;  // samples of row `lane`
        const int upto = wave_inclusive_scan(mine);
        for (int s0 = 0; s0 < p.per; s0 += 64) {
            const int s = un.z * p.per + s0 + lane;  // this lane's sample
            int row = -1, idx = 0;
            for (int r = 0; r < p.V; r++) {
                const int before = __shfl(upto - mine, r, 64), n = __shfl(mine, r, 64);
                if (s >= before && s < before + n) { row = r; idx = s - before; }
            }
            const bool live = row >= 0 && s0 + lane < p.per;
            const int32_t lo_s = __shfl(lo, max(row, 0), 64);
            const int32_t c = live ? a.colidx[lo_s + (idx + 1) * p.stride - 1] : 0;
            int rank = idx, below[ROWS];
    #pragma unroll
            for (int r0 = 0; r0 < ROWS; r0 += G) {
                int32_t base[G];
                int m[G], most = 0;
    #pragma unroll
                for (int g = 0; g < G; g++) {
                    const int r = r0 + g;
                    m[g] = __shfl(mine, min(r, 63), 64);
                    base[g] = __shfl(lo, min(r, 63), 64) + p.stride - 1;
                    if (!live || r == row || r >= p.V) m[g] = 0;
                    below[r] = 0;
                    most = max(most, m[g]);
                }
                for (; __any(most > 0); most >>= 1) {  // halves until every row's samples are told apart
    #pragma unroll
                    for (int g = 0; g < G; g++) {
                        const int half = m[g] >> 1;
                        const int32_t v = m[g] > 0 ? a.colidx[base[g] + (below[r0 + g] + half) * p.stride] : 0;
                        const bool less = m[g] > 0 && (v < c || (v == c && r0 + g < row));
                        below[r0 + g] += less ? half + 1 : 0;
                        m[g] = less ? m[g] - half - 1 : half;
                    }
                }
    #pragma unroll
                for (int g = 0; g < G; g++) rank += below[r0 + g];
            }
            const int q = rank / p.per;
            const bool starts = live && rank == q * p.per && q > 0 && q < un.w;
            if (!__any(starts)) continue;
    #pragma unroll
            for (int r0 = 0; r0 < ROWS; r0 += G) {
                int32_t at[G], end[G];
    #pragma unroll
                for (int g = 0; g < G; g++) {
                    const int r = min(r0 + g, 63);
                    const int n = r == row ? idx : below[r0 + g];  // the last of them may be the column itself (a row before `row`)
                    at[g] = __shfl(lo, r, 64) + max(n * p.stride - 1, 0);
                    end[g] = min(at[g] + p.stride + 1, __shfl(hi, r, 64));
                    if (!starts || r0 + g >= p.V) end[g] = at[g];
                }
                for (int step = 1; step < 2 * p.stride; step <<= 1) {
    #pragma unroll
                    for (int g = 0; g < G; g++) {
                        const int32_t mid = at[g] + ((end[g] - at[g]) >> 1);
                        const bool some = at[g] < end[g], less = some && a.colidx[mid] < c;
                        if (less) at[g] = mid + 1; else if (some) end[g] = mid;
                    }
                }
    #pragma unroll
                for (int g = 0; g < G; g++)
                    if (starts && r0 + g < p.V) start[(int64_t)(u - un.z + q) * p.V + r0 + g] = at[g];
            }
        }
    }
}

// A row of a unit: window wl of the unit, row r of the window.  The lane that holds it says where it stands among
// the unit's rows.
struct UnitRows {
    int32_t row_lo;       // the row's first entry
    int32_t lo, len;      // the unit's share of the row
    int begin;            // its first entry among the unit's, row after row in lane order
    int total;            // entries of the unit
};
// What has to be read for that, as it stands in memory.
struct UnitRowLoads {
    int32_t lo, hi, piece_lo, piece_hi;
};
__device__ __forceinline__ bool unit_row_live(const CsrView &a, const UnitPlan &p, const int4 &un, int wl, int r)
{
    return wl < un.y && r < p.V && ((int64_t)un.x + wl) * p.V + r < a.M;
}
__device__ __forceinline__ UnitRowLoads load_unit_rows(const CsrView &a, const UnitPlan &p, const int4 &un, int u, int wl, int r, const int32_t *__restrict__ piece_start)
{
    UnitRowLoads l{0, 0, 0, 0};
    if (!unit_row_live(a, p, un, wl, r)) return l;
    const int64_t row = ((int64_t)un.x + wl) * p.V + r;
    l.lo = a.rowptr[row];
    l.hi = a.rowptr[row + 1];
    if (un.w > 1) {
        if (un.z > 0) l.piece_lo = piece_start[(int64_t)u * p.V + r];
        if (un.z + 1 < un.w) l.piece_hi = piece_start[((int64_t)u + 1) * p.V + r];
    }
    return l;
}
__device__ __forceinline__ UnitRows unit_rows(const CsrView &a, const UnitPlan &p, const int4 &un, const UnitRowLoads &l, int wl, int r, bool &bad)
{
    UnitRows x;
    x.row_lo = min(max(l.lo, 0), a.nnz);  // (clamped as by row_range)
    int32_t hi = min(max(l.hi, x.row_lo), a.nnz);
    x.lo = x.row_lo;
    if (un.w > 1 && unit_row_live(a, p, un, wl, r)) {
        const int32_t end = hi;
        if (un.z + 1 < un.w) hi = l.piece_hi;
        if (un.z > 0) x.lo = l.piece_lo;
        if (x.lo < x.row_lo || hi < x.lo || hi > end) {  // columns that do not ascend
            bad = true;
            x.lo = hi = x.row_lo;
        }
    }
    x.len = hi - x.lo;
    int upto = wave_inclusive_scan(x.len);
    x.total = __builtin_amdgcn_readlane(upto, 63);  // known to be the same for all lanes: what depends on it are branches, not masks
    if (x.total > kUnitEntries) {  // columns that do not ascend, again: nothing of this unit is used
        bad = true;
        x.len = x.total = upto = 0;
    }
    x.begin = upto - x.len;
    return x;
}

// Ranks: info[p] = rank of entry p's vector among the vectors of its unit | its row in the unit << 9 (row r of window
// wl: wl * 2^lv + r); count[u] = vectors of unit u; win_at[w] = {the unit window w begins in, vectors of that
// unit before it}.  Checks the columns (err |= 2).
//
// A vector is a number (window, column less the unit's smallest one), and its rank is how many different such numbers are smaller: what a
// trie tells whose nodes are 32-bit masks.  The entries set the bits of the top level, up to 2^kTopBits of them; the number of set
// bits before an entry's is its node on the next level, five bits further down, and on the last level it is the rank.  A level
// costs an entry one LDS operation to set its bit and two to count, about twelve instructions whatever the rows are, and a prefix sum over its
// at most 512 nodes.  Units of short windows of a matrix with 2^20 columns take three levels, pieces of hubs one or two.  What bounds it is
// the issue of instructions (530 for the 314 entries of a unit on average of R-MAT of 1 M rows, 31 M entries; a merge of the rows
// in log2(V) rounds of binary searches took 1450) and what a wavefront waits for, so the chip's wavefronts walk the units with the
// next ones' records and row pointers under way: 238 -> 119 us, 190 MB; the vector units are busy 70 % of that, LDS 51 %.  (Nodes of
// 64 bits, six bits a level: 770 instructions, 6 KB of LDS and 183 us.)
constexpr int kTopBits = 14, kDigitBits = 5;
constexpr int kFewEntries = 8;  // as many are compared one by one (16 M rows with 1 M entries, four a unit: by the trie 193 us, so 147)
constexpr int kRankGrid = 32 * 256;  // wavefronts that the chip holds at once
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8))) k_unit_rank(CsrView a, UnitPlan p, int64_t K, const int4 *__restrict__ units, const int *__restrict__ n_units,
                                                  const int32_t *__restrict__ piece_start, uint16_t *__restrict__ info, int *__restrict__ count,
                                                  int2 *__restrict__ win_at, int *__restrict__ err)
{
    constexpr int NCH = kUnitEntries / 64, PER = kUnitEntries / 64;  // entries and nodes of a lane
    static_assert((1 << kTopBits) / 32 <= kUnitEntries && PER == 8, "nodes of the top level; sixteen-byte accesses");
    __shared__ __attribute__((aligned(16))) uint32_t node[kUnitEntries];
    __shared__ __attribute__((aligned(16))) uint16_t before[kUnitEntries];  // set bits of the level before a node's
    __shared__ int2 row_of[kUnitRows];      // rows with entries, in order: {row, what to add to an entry's place in the unit}
    __shared__ int32_t sh_lo[kUnitRows];    // the latter by row
    __shared__ uint32_t opens[2 * NCH];     // a bit per entry that opens a row
    __shared__ int win_first[kMaxUnitWindows];
    int lane = threadIdx.x;
    const int wl = lane >> p.lv, r = lane & ((1 << p.lv) - 1);
    if (*err & 1) return;  // malformed row pointers: the records are not there
    const int n_all = *n_units;
    // a unit's record, by a vector load (a scalar one under way would be waited for by every use of LDS)
    auto record = [&](uint32_t u) -> int4 {
        uint32_t at = min(u, (uint32_t)n_all - 1);
        asm volatile("" : "+v"(at));
        return units[at];
    };
    auto uniform = [](const int4 &v) -> int4 {
        return make_int4(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y), __builtin_amdgcn_readfirstlane(v.z), __builtin_amdgcn_readfirstlane(v.w));
    };
    // The record of the unit after next and the row pointers of the next one are read while a unit is ranked.
    if ((int)blockIdx.x >= n_all) return;
    int4 un = uniform(record(blockIdx.x)), coming = record(blockIdx.x + gridDim.x);
    UnitRowLoads loads = load_unit_rows(a, p, un, blockIdx.x, wl, r, piece_start);
    for (uint32_t u = blockIdx.x; u < (uint32_t)n_all; u += gridDim.x) {
        bool bad = false;
        asm volatile("" : "+v"(lane));  // (numbers that follow from it are not kept from unit to unit)
        const UnitRows x = unit_rows(a, p, un, loads, wl, r, bad);
        int E = x.total;
        if (lane < 2 * NCH) opens[lane] = 0;
        if (lane < kMaxUnitWindows) win_first[lane] = INT32_MAX;
        FS_WAVE_SYNC();
        sh_lo[lane] = x.lo - x.begin;
        const uint64_t with = __ballot(x.len > 0);
        if (x.len > 0) {
            row_of[__builtin_amdgcn_mbcnt_hi((uint32_t)(with >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)with, 0))] = make_int2(lane, x.lo - x.begin);
            atomicOr(&opens[x.begin >> 5], 1u << (x.begin & 31));
        }
        FS_WAVE_SYNC();
        uint32_t col[NCH];
        int row[NCH];
        uint64_t first_of[NCH];  // entries that open a row, the same for all lanes
        int2 of[NCH];
        const int opening_words = (int)opens[lane & (2 * NCH - 1)];
        int rows_so_far = 0;
        FS_EACH(h) {  // the reads of all of a lane's entries are under way together: no branches
            first_of[h] = (uint32_t)__builtin_amdgcn_readlane(opening_words, 2 * h) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane(opening_words, 2 * h + 1) << 32;
            // the row of entry e is the one that the last opening at e or before it begins
            const uint64_t later = first_of[h] >> 1;
            const int k = rows_so_far - 1 + (int)(first_of[h] & 1);
            rows_so_far += __popcll(first_of[h]);
            of[h] = row_of[max((int)__builtin_amdgcn_mbcnt_hi((uint32_t)(later >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)later, (uint32_t)k)), 0)];
        } FS_EACH_END;
        FS_EACH(h) {  // every load of the unit is on its way before the first use
            row[h] = of[h].x;
            col[h] = 0;
            if (64 * h < E) col[h] = (uint32_t)a.colidx[of[h].y + 64 * h + min(lane, E - 1 - 64 * h)];
        } FS_EACH_END;
        if (un.w > 1 && x.len > 0 && x.lo > x.row_lo && a.colidx[x.lo - 1] >= a.colidx[x.lo]) bad = true;  // across the cut
        FS_WAIT_LOADS();
        const int4 next = uniform(coming);
        loads = load_unit_rows(a, p, next, (int)min(u + gridDim.x, (uint32_t)n_all - 1), wl, r, piece_start);
        coming = record(u + 2 * gridDim.x);
        uint32_t last = 0, least = INT32_MAX, most = 0;  // last: the previous 64 entries' last column
        FS_EACH(h) {
            if (64 * h < E) {
                // (lanes past the last entry hold its column once more, and are not looked at)
                const uint32_t c = col[h], prev = (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)c, 0x138, 0xF, 0xF, false);  // wave_shr:1
                last = (uint32_t)__builtin_amdgcn_readlane((int)c, 63);
                const bool opening = __builtin_amdgcn_inverse_ballot_w64(first_of[h]);
                if (lane < E - 64 * h && (c >= (uint32_t)K || (!opening && prev >= c))) bad = true;
                least = min(least, c);
                most = max(most, c);
            }
        } FS_EACH_END;
        if (__ballot(bad)) {  // what follows takes numbers from the columns: nothing of this unit is used
            if (lane == 0) atomicOr(err, 2);
            E = 0;
        }
        E = __builtin_amdgcn_readfirstlane(E);
        int vectors = 0;
        int at[NCH];  // an entry's node, at last its rank
        FS_EACH(h) at[h] = 0; FS_EACH_END;
        if (E <= kFewEntries) {  // one after the other
            const uint64_t mine = (uint64_t)(uint32_t)(row[0] >> p.lv) << 32 | col[0];
            auto number = [&](int j) -> uint64_t {
                return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), j) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)mine, j);
            };
            bool leads = lane < E;  // no earlier entry of the same vector
            for (int j = 0; j + 1 < E; j++) leads = leads && !(lane > j && number(j) == mine);
            const uint64_t led = __ballot(leads);
            vectors = __popcll(led);
            for (uint64_t m = led; m; m &= m - 1) at[0] += number(__builtin_ctzll(m)) < mine ? 1 : 0;
        } else {
            // (columns are below 2^31: signed comparisons do)
            least = (uint32_t)__builtin_amdgcn_readlane(wave_scan((int)least, INT32_MAX, [](int a, int b) { return min(a, b); }), 63);
            const uint32_t span = (uint32_t)__builtin_amdgcn_readlane(wave_scan((int)most, 0, [](int a, int b) { return max(a, b); }), 63) - least;
            const int col_bits = 32 - __builtin_clz(span | 1), win_bits = un.y == 1 ? 0 : 32 - __builtin_clz(un.y - 1);
            const int below = max(col_bits + win_bits - kTopBits + kDigitBits - 1, 0) / kDigitBits;  // levels below the top one
            const int top = col_bits - kDigitBits * below;                                          // a column's bits on the top level
            // One level: bit(h) says which bit of its node an entry sets.  Returns how many are set.
            auto walk = [&](auto bit) -> int {
                fs_u4 *mine = reinterpret_cast<fs_u4 *>(node + lane * PER);
                mine[0] = mine[1] = fs_u4{0u, 0u, 0u, 0u};
                FS_WAVE_SYNC();
                FS_EACH(h) {
                    if (lane < E - 64 * h) atomicOr(node + at[h], 1u << (bit(h) & 31));
                } FS_EACH_END;
                FS_WAVE_SYNC();
                int c[PER + 1];
                c[0] = 0;
                const fs_u4 m[2] = {mine[0], mine[1]};
#pragma unroll
                for (int k = 0; k < PER; k++) c[k + 1] = c[k] + __popc(m[k / 4][k % 4]);
                const int upto = wave_inclusive_scan(c[PER]), from = upto - c[PER];
                fs_u4 o;
#pragma unroll
                for (int k = 0; k < PER / 2; k++) o[k] = (uint32_t)(from + c[2 * k]) | (uint32_t)(from + c[2 * k + 1]) << 16;
                *reinterpret_cast<fs_u4 *>(before + lane * PER) = o;
                FS_WAVE_SYNC();
                FS_EACH(h) {
                    if (64 * h < E) {
                        asm volatile("" : "+v"(col[h]), "+v"(at[h]));  // worked out again, not kept from above
                        at[h] = before[at[h]] + __popc(node[at[h]] & ((1u << (bit(h) & 31)) - 1));
                    }
                } FS_EACH_END;
                FS_WAVE_SYNC();
                return __builtin_amdgcn_readlane(upto, 63);
            };
            auto on_top = [&](int h) -> uint32_t { return ((uint32_t)(row[h] >> p.lv) << top) + (col[h] >> (kDigitBits * below)); };
            FS_EACH(h) {
                if (64 * h < E) {
                    col[h] -= least;
                    at[h] = (int)(on_top(h) >> 5);
                }
            } FS_EACH_END;
            vectors = walk(on_top);
            for (int shift = kDigitBits * (below - 1); shift >= 0; shift -= kDigitBits) vectors = walk([&](int h) -> uint32_t { return col[h] >> shift; });
        }
        FS_EACH(h) {
            if (lane < E - 64 * h) {
                asm volatile("" : "+v"(row[h]));  // read again, not kept
                info[sh_lo[row[h]] + 64 * h + lane] = (uint16_t)(at[h] | (row[h] << 9));
                if (__builtin_amdgcn_inverse_ballot_w64(first_of[h])) atomicMin(&win_first[row[h] >> p.lv], at[h]);  // a window's first vector is some row's first entry
            }
        } FS_EACH_END;
        if (lane == 0) count[u] = vectors;
        FS_WAVE_SYNC();
        if (un.z == 0) {
            const int mine = lane < kMaxUnitWindows ? win_first[lane] : INT32_MAX;
            const uint64_t seen = __ballot(mine != INT32_MAX);  // windows with entries
            if (lane < un.y) {
                const uint64_t after = seen >> lane;  // an empty window begins where the next one with entries does
                win_at[un.x + lane] = make_int2((int)u, after ? win_first[lane + __builtin_ctzll(after)] : vectors);
            }
        }
        un = next;
        FS_WAVE_SYNC();
    }
}

// Every unit's first vector (first_vec[n_units]: the number of vectors), the window pointers, and the block slots of every workgroup's
// windows.  A workgroup takes `tiles` times kWindowThreads windows, which begin with a unit, and scans their units itself; what lies before them it
// adds up from the units' counts, or from `sums`, the counts of kScanTile units each (as they are, or scanned, of which there may be any
// number).  One launch instead of three: the scans of a small conversion were single workgroups, 4 us each and as much between them.
constexpr int kWindowThreads = 1024;
__global__ void __launch_bounds__(kWindowThreads) k_win_ptr(const int2 *__restrict__ win_at, const int *__restrict__ count, const int *__restrict__ sums, bool scanned,
                                                            const int *__restrict__ n_units, int64_t W, int KB, int tiles, int *first_vec,
                                                            int32_t *__restrict__ win_ptr, int *__restrict__ slots, int *__restrict__ misc)
{
    const int64_t w0 = (int64_t)blockIdx.x * tiles * kWindowThreads, w1 = min(w0 + (int64_t)tiles * kWindowThreads, W);
    if (W == 0 || (misc[0] & 1)) {  // no rows, or malformed row pointers: nothing was counted
        for (int64_t w = w0 + threadIdx.x; w < w1; w += kWindowThreads) win_ptr[w] = 0;
        if (w1 == W && threadIdx.x == 0) win_ptr[W] = 0;
        if (threadIdx.x == 0) slots[blockIdx.x] = (int)(w1 - w0);
        return;
    }
    const int u0 = win_at[w0].x, u1 = w1 < W ? win_at[w1].x : *n_units;
    int from = 0, mine = 0;
    if (sums) {
        const int t = u0 / kScanTile;
        from = t * kScanTile;
        if (scanned) mine = threadIdx.x == 0 ? sums[t] : 0;
        else
            for (int k = threadIdx.x; k < t; k += kWindowThreads) mine += sums[k];
    }
    for (int i0 = from + threadIdx.x * 8; i0 < u0; i0 += 8 * kWindowThreads) {
        int v[8];
        scan_load8(count, i0, u0, v);
#pragma unroll
        for (int k = 0; k < 8; k++) mine += v[k];
    }
    int before[1] = {mine};
    block_sum<kWindowThreads>(before);
    int ahead = before[0];
    for (int u = u0; u < u1; u += kWindowThreads) {
        const int i = u + (int)threadIdx.x, c = i < u1 ? count[i] : 0;
        int here;
        const int first = ahead + block_exclusive_scan<kWindowThreads>(c, &here);
        if (i < u1) first_vec[i] = first;
        ahead += here;
    }
    if (w1 == W && threadIdx.x == 0) {
        first_vec[u1] = ahead;
        win_ptr[W] = ahead;
        misc[1] = ahead;
    }
    __syncthreads();  // first_vec is read back by other threads than wrote it
    auto ptr = [&](int64_t w) -> int32_t {
        if (w >= w1) return ahead;
        const int2 at = win_at[w];
        return first_vec[at.x] + at.y;
    };
    int made[1] = {0}, longest = 0;
    for (int64_t w = w0 + threadIdx.x; w < w1; w += kWindowThreads) {
        const int32_t q = ptr(w);
        win_ptr[w] = q;
        const int n = max(1, (ptr(w + 1) - q + KB - 1) / KB);
        made[0] += n;
        longest = max(longest, n);
    }
    longest = wave_scan(longest, 0, [](int a, int b) { return max(a, b); });
    __shared__ int most[kWindowThreads / 64];
    if ((threadIdx.x & 63) == 63) most[threadIdx.x >> 6] = longest;
    block_sum<kWindowThreads>(made);  // (with its barriers)
    if (threadIdx.x == 0) {
        slots[blockIdx.x] = made[0];
        for (int k = 0; k < kWindowThreads / 64; k++) longest = max(longest, most[k]);
        atomicMax(&misc[2], longest);
    }
}

// What the second kernel writes.  vals null: pattern only (the value array is cleared beforehand); packed_* null: not wanted.
struct PlaceOut {
    int32_t *vec_col;
    uint32_t *vec_mask;
    int32_t *csr_to_slot;
    uint16_t *vals_blk;
    int4 *blk_desc;
    int32_t *row_base;
    uint32_t *row_bits;
    int32_t *packed_ofs;
    uint8_t *packed_m8;
    uint16_t *packed_m16;
    uint16_t *packed_vals;
    uint16_t *tail;  // the elements behind the value array that have to be zero
    int n_tail;
    int n_blocks;
};

// LDS of k_unit_place: a unit's vectors (columns and masks, later its share of the value array), then two tables with an
// element per block of 32 vectors and row.
constexpr int kTileVectors = 256;
inline size_t place_vector_bytes(int V) { return (size_t)(V * 2 * kTileVectors > kUnitEntries * 8 ? V * 2 * kTileVectors : kUnitEntries * 8); }
inline size_t place_lds_bytes(int V, int KB) { return place_vector_bytes(V) + (KB == 32 ? (size_t)(kUnitEntries / 32 + kMaxUnitWindows + 2) * V * 8 : 0); }

// Everything of the format that belongs to a unit's entries, vectors and blocks.  KB32: blocks of 32 vectors, the width
// the compute kernels take: their rows' occupancy and CSR positions are written too.  A block that a hub window's pieces
// share gets its values from k_shared_blocks.
template <bool KB32, int VT>  // VT: rows per window, or 0 for those without an instantiation of their own
__global__ void __launch_bounds__(64) k_unit_place(int block0, CsrView a, UnitPlan p, int KB, int64_t vec_bytes, const int4 *__restrict__ units,
                                                   const int32_t *__restrict__ piece_start, const uint16_t *__restrict__ info,
                                                   const int *__restrict__ first_vec, const int32_t *__restrict__ win_ptr, const int *__restrict__ blk_ptr,
                                                   const uint16_t *__restrict__ vals, PlaceOut out)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ int begin[kUnitRows + 1];
    __shared__ int32_t sh_lo[kUnitRows];
    __shared__ int32_t row_start[kUnitRows];
    __shared__ int32_t wp[kMaxUnitWindows + 1], bp[kMaxUnitWindows + 1];
    if constexpr (VT > 0) {
        p.V = VT;
        p.lv = 31 - __builtin_clz(VT);
    }
    const int u = block0 + blockIdx.x, lane = threadIdx.x, V = p.V;
    if (u == 0) {
        for (int i = lane; i < out.n_tail; i += 64) out.tail[i] = 0;
        if (out.packed_ofs && lane == 0) out.packed_ofs[out.n_blocks] = a.nnz;
    }
    if constexpr (KB32) KB = 32;
    const int4 un = units[u];
    bool bad = false;
    const int my_wl = lane >> p.lv, my_r = lane & ((1 << p.lv) - 1);
    const UnitRows x = unit_rows(a, p, un, load_unit_rows(a, p, un, u, my_wl, my_r, piece_start), my_wl, my_r, bad);
    const int E = x.total;
    const int f = first_vec[u], n = first_vec[u + 1] - f;
    begin[lane] = x.begin;
    sh_lo[lane] = x.lo - x.begin;
    if (lane <= un.y) {
        wp[lane] = win_ptr[un.x + lane];
        bp[lane] = blk_ptr[un.x + lane];
    }
    FS_WAVE_SYNC();
    const bool hub = un.w > 1;
    const int o = f - wp[0];                 // vectors of the window before the unit (hub windows only, else 0)
    const int b_lo = o / KB;                 // the window's block that the unit's first vector lies in
    const int n_w0 = wp[1] - wp[0];
    // tables: blocks of the unit, window after window (of a hub window those the unit's vectors lie in)
    const int n_t = hub ? (n > 0 ? (o + n - 1) / KB - b_lo + 1 : 0) : bp[un.y] - bp[0];
    int *col_buf = reinterpret_cast<int *>(lds);
    uint32_t *mask_buf = reinterpret_cast<uint32_t *>(lds) + kUnitEntries;
    uint32_t *bits = reinterpret_cast<uint32_t *>(lds + vec_bytes);  // occupancy of a block's row
    int32_t *packed_at = reinterpret_cast<int32_t *>(bits + (size_t)n_t * V);
    for (int i = lane; i < n; i += 64) mask_buf[i] = 0;
    if constexpr (KB32) {
        for (int i = lane; i < n_t * V; i += 64) bits[i] = 0;
    }
    FS_WAVE_SYNC();

    // blocks whose vectors all lie in the unit (hub windows; of other units all do)
    const int own_lo = hub ? (o + KB - 1) / KB : 0, own_hi = hub ? (o + n == n_w0 ? (n_w0 + KB - 1) / KB : (o + n) / KB) : INT32_MAX;
    // the unit's entries, up to eight per lane: every load is on its way before the first use
    constexpr int NCH = kUnitEntries / 64;
    int32_t pos[NCH], col[NCH];
    int code[NCH];  // rank | row << 9
    int val[NCH];
    const uint16_t *val_src = vals ? vals : info;  // (something to read in a pattern-only conversion)
    FS_EACH(h) {
        pos[h] = col[h] = code[h] = 0;
        val[h] = 0;
        if (64 * h < E) {
            const int e = min(64 * h + lane, E - 1);
            int i = 0;  // (whole windows: their rows follow each other, and the code names the row)
            if (hub)
                for (int w = 1 << p.lv >> 1; w > 0; w >>= 1) i += begin[i + w] <= e ? w : 0;
            pos[h] = sh_lo[i] + e;
            code[h] = info[pos[h]];
            col[h] = a.colidx[pos[h]];
            val[h] = val_src[pos[h]];
        }
    } FS_EACH_END;
    FS_WAIT_LOADS();
    // of an entry: window of the unit, row, vector of the window, block of the window
    auto place = [&](int cd, int &wl, int &row, int &kw, int &b) {
        wl = (cd >> 9) >> p.lv;
        row = (cd >> 9) & ((1 << p.lv) - 1);
        kw = f + (cd & 511) - wp[wl];
        b = kw / KB;
    };
    FS_EACH(h) {
        if (64 * h + lane < E) {
            int wl, row, kw, b;
            place(code[h], wl, row, kw, b);
            col_buf[code[h] & 511] = col[h];  // the same from every entry of the vector
            atomicOr(&mask_buf[code[h] & 511], 1u << row);
            if constexpr (KB32) atomicOr(&bits[(bp[wl] - bp[0] + b - b_lo) * V + row], 1u << (kw - b * KB));
        }
    } FS_EACH_END;
    FS_WAVE_SYNC();
    for (int i = lane; i < n; i += 64) {
        const uint32_t m = mask_buf[i];
        out.vec_col[f + i] = col_buf[i];
        out.vec_mask[f + i] = m;
        if (out.packed_m8) out.packed_m8[f + i] = (uint8_t)m;
        if (out.packed_m16) out.packed_m16[f + i] = (uint16_t)m;
    }
    // Block tables, 64 (block, row) pairs at a time, in the order the format keeps them.
    auto window_of_block = [&](int t) -> int {  // of the unit's block t
        int w = 0;
        if (un.y > 1)
            for (int h = kMaxUnitWindows >> 1; h > 0; h >>= 1) w += w + h < un.y && bp[w + h] - bp[0] <= t ? h : 0;
        return w;
    };
    if constexpr (KB32) {
        row_start[lane] = x.lo;
        // entries of the window that earlier pieces hold
        int ahead = x.lo - x.row_lo;
        for (int h = 1; h < (1 << p.lv); h <<= 1) ahead += __shfl_xor(ahead, h, 64);
        int packed = __shfl(x.row_lo, 0, 64) + __shfl(ahead, 0, 64);  // in packed order entries go block by block, row by row
        const int n_pairs = n_t * V;
        FS_WAVE_SYNC();
        for (int i0 = 0; i0 < n_pairs; i0 += 64) {
            const int i = i0 + lane;
            const uint32_t m = i < n_pairs ? bits[i] : 0u;
            const int cnt = __popc(m);
            const int upto = wave_inclusive_scan(cnt);
            if (i < n_pairs) packed_at[i] = packed + upto - cnt;
            packed += __shfl(upto, 63, 64);
        }
        FS_WAVE_SYNC();
        for (int i0 = 0; i0 < n_pairs; i0 += 64) {
            const int i = i0 + lane;
            if (i < n_pairs) {
                const int t = i / V, row = i - t * V;
                const int wl = window_of_block(t), first_t = bp[wl] - bp[0];
                int before = 0;  // the row's entries in the window's earlier blocks of the unit
                for (int k = first_t; k < t; k++) before += __popc(bits[k * V + row]);
                const int b = b_lo + t - first_t;
                if (b * KB >= o) {  // the block starts here
                    const int64_t at = (int64_t)(bp[wl] + b) * V + row;
                    out.row_base[at] = row_start[(wl << p.lv) + row] + before;
                    if (b < own_hi) out.row_bits[at] = bits[i];
                }
            }
        }
    }
    for (int t = lane; t < n_t; t += 64) {
        const int wl = window_of_block(t), b = b_lo + t - (bp[wl] - bp[0]);
        if (b * KB >= o) {
            const int n_w = wp[wl + 1] - wp[wl], kb = max(0, min(KB, n_w - b * KB));
            out.blk_desc[bp[wl] + b] = make_int4(wp[wl] + b * KB, kb | ((b + 1) * KB >= n_w ? 256 : 0) | (b == 0 ? 512 : 0), un.x + wl, 0);
            if (KB32 && out.packed_ofs) out.packed_ofs[bp[wl] + b] = packed_at[t * V];
        }
    }
    FS_WAVE_SYNC();
    // The unit's share of the value array, put together where the columns were, kTileVectors vectors at a time: zeros,
    // then the entries, then the copy out; after it the packed values, in their order.
    const int v_lo = hub ? min(own_lo * KB, n_w0) + wp[0] : f;
    const int v_hi = hub ? max(min(own_hi * KB, n_w0) + wp[0], v_lo) : f + n;
    const int A = V * v_lo, n_el = V * (v_hi - v_lo);
    int slot[NCH];  // relative to A; negative: not the unit's own
    int pk[NCH];    // place in packed order
    const int pk_lo = KB32 && out.packed_vals && v_lo < v_hi ? packed_at[(own_lo - b_lo) * V] : 0;
    int n_pk = 0;
    FS_EACH(h) {
        slot[h] = -1;
        pk[h] = 0;
        if (64 * h < E) {
            bool own = false;
            if (64 * h + lane < E) {
                int wl, row, kw, b;
                place(code[h], wl, row, kw, b);
                const int c = kw - b * KB, kb = min(KB, wp[wl + 1] - wp[wl] - b * KB);
                const int at = V * (wp[wl] + b * KB) + row * kb + c;
                out.csr_to_slot[pos[h]] = at;
                own = b >= own_lo && b < own_hi;
                if (own) slot[h] = at - A;
                if (KB32 && own && out.packed_vals) {
                    const int i = (bp[wl] - bp[0] + b - b_lo) * V + row;
                    pk[h] = packed_at[i] + __popc(bits[i] & ((1u << c) - 1)) - pk_lo;
                }
            }
            n_pk += __popcll(__ballot(own));
        }
    } FS_EACH_END;
    if (!vals) return;
    uint16_t *tile = reinterpret_cast<uint16_t *>(lds);
    for (int e0 = 0; e0 < n_el; e0 += kTileVectors * V) {
        const int m = min(n_el - e0, kTileVectors * V);
        for (int i = lane * 8; i < m; i += 512) *reinterpret_cast<fs_u4 *>(tile + i) = fs_u4{0u, 0u, 0u, 0u};
        FS_WAVE_SYNC();
        FS_EACH(h) {
            if (64 * h < E && slot[h] >= e0 && slot[h] < e0 + m) tile[slot[h] - e0] = (uint16_t)val[h];
        } FS_EACH_END;
        FS_WAVE_SYNC();
        uint16_t *dst = out.vals_blk + A + e0;
        if (V % 8 == 0) {
            for (int i = lane * 8; i < m; i += 512) *reinterpret_cast<fs_u4 *>(dst + i) = *reinterpret_cast<const fs_u4 *>(tile + i);
        } else if (V % 4 == 0) {
            for (int i = lane * 4; i < m; i += 256) *reinterpret_cast<uint2 *>(dst + i) = *reinterpret_cast<const uint2 *>(tile + i);
        } else {
            for (int i = lane; i < m; i += 64) dst[i] = tile[i];
        }
        FS_WAVE_SYNC();
    }
    if (KB32 && out.packed_vals) {
        FS_EACH(h) {
            if (64 * h < E && slot[h] >= 0) tile[pk[h]] = (uint16_t)val[h];
        } FS_EACH_END;
        FS_WAVE_SYNC();
        for (int i = lane; i < n_pk; i += 64) out.packed_vals[pk_lo + i] = tile[i];
    }
}

// A block that more than one piece of a hub window reaches into is finished by the first piece that begins inside it.  Its
// vectors, and the CSR position of each row's first entry in it, are in place.  A unit's record, its first vector and the one of the unit
// before it; from them the block, its first vector and its width; xb: the block slot, or -1 (none).
struct SharedBlock {
    int xb, s, kb;
};
__device__ __forceinline__ SharedBlock shared_block(bool live, int KB, const int4 &un, int first, int first_before, int f_w, int f_next, int slot0)
{
    const int n_w = f_next - f_w, o = first - f_w, b = o / KB;
    const bool shared = live && un.w > 1 && un.z > 0 && o > b * KB && o < n_w && first_before - f_w <= b * KB;
    return SharedBlock{shared ? slot0 + b : -1, f_w + b * KB, shared ? min(KB, n_w - b * KB) : 0};
}

// Blocks of 32 vectors: half a wavefront per unit, so that its two blocks wait for memory together (four of them need the registers of
// the other wavefronts: 51 us).  A block's values pass through LDS, eight rows at a time, and leave in sixteen-byte pieces.  What bounds it is
// the chain record -> window -> masks -> values of short wavefronts: R-MAT of 1 M rows, 100 k units, values stored row by row and one by
// one 51 us, now 45.
constexpr int kSharedPerWave = 2;  // units a wavefront looks at
constexpr int kSharedStage = 8 * 32;  // elements of eight rows of a block
__device__ __forceinline__ void finish_shared_blocks(int64_t u0, int n_units, int V, const int4 *__restrict__ units, const int *__restrict__ first_vec,
                                                     const int32_t *__restrict__ win_ptr, const int *__restrict__ blk_ptr,
                                                     const uint16_t *__restrict__ vals, const PlaceOut &out, uint16_t *stage /* 2 * kSharedStage of this half */)
{
    const int lane = threadIdx.x & 63, half = lane & 32, c = lane & 31;
    const int u = (int)min(u0 + (half >> 5), (int64_t)n_units - 1);
    const int4 un = units[u];
    const SharedBlock sb = shared_block(u0 + (half >> 5) < n_units, 32, un, first_vec[u], first_vec[max(u - 1, 0)], win_ptr[un.x], win_ptr[un.x + 1], blk_ptr[un.x]);
    if (!__ballot(sb.xb >= 0)) return;
    const uint32_t m = c < sb.kb ? out.vec_mask[sb.s + c] : 0u;  // (nothing stored where there is no block)
    const int32_t base = sb.xb >= 0 && c < V ? out.row_base[(int64_t)sb.xb * V + c] : 0;
    int32_t packed = sb.xb >= 0 && out.packed_vals ? out.packed_ofs[sb.xb] : 0;
    const uint32_t below = (1u << c) - 1;
    for (int r0 = 0; r0 < V; r0 += 8) {  // eight rows' loads together
        uint16_t v[8];
        uint32_t mine = 0;  // occupancy of row r0 + c, in the first eight lanes
#pragma unroll
        for (int g = 0; g < 8; g++) {
            const int r = r0 + g;
            const bool has = r < V && ((m >> r) & 1u);
            const uint64_t both = __ballot(has);
            const uint32_t row = (uint32_t)(half ? both >> 32 : both);
            if (c == g) mine = row;
            const int32_t q = __shfl(base, half + min(r, 31), 64) + __popc(row & below);
            v[g] = has && vals ? vals[q] : (uint16_t)0;
        }
        const int rows = min(V - r0, 8);
        if (sb.xb >= 0 && c < rows) out.row_bits[(int64_t)sb.xb * V + r0 + c] = mine;
        if (!vals) continue;
        int n = 0;  // stored values so far
#pragma unroll
        for (int g = 0; g < 8; g++) {
            const uint32_t row = __shfl(mine, half + g, 64);
            if (g < rows && c < sb.kb) stage[g * sb.kb + c] = v[g];
            if ((row >> c) & 1u) stage[kSharedStage + n + __popc(row & below)] = v[g];
            n += __popc(row);
        }
        FS_WAVE_SYNC();
        uint16_t *dst = out.vals_blk + (int64_t)V * sb.s + r0 * sb.kb;
        if (V % 8 == 0) {
            if (c * 8 < rows * sb.kb) *reinterpret_cast<fs_u4 *>(dst + c * 8) = *reinterpret_cast<const fs_u4 *>(stage + c * 8);
        } else if (V % 4 == 0) {
            for (int i = c * 4; i < rows * sb.kb; i += 128) *reinterpret_cast<uint2 *>(dst + i) = *reinterpret_cast<const uint2 *>(stage + i);
        } else {
            for (int i = c; i < rows * sb.kb; i += 32) dst[i] = stage[i];
        }
        if (out.packed_vals)
            for (int i = c; i < n; i += 32) out.packed_vals[packed + i] = stage[kSharedStage + i];
        packed += n;
        FS_WAVE_SYNC();
    }
}

constexpr int kSharedWaves = 4;  // per workgroup: they share nothing, but there are a quarter as many to start
__global__ void __launch_bounds__(64 * kSharedWaves) __attribute__((amdgpu_waves_per_eu(8))) k_shared_blocks(int block0, int V, const int4 *__restrict__ units, int n_units, const int *__restrict__ first_vec,
                                                      const int32_t *__restrict__ win_ptr, const int *__restrict__ blk_ptr,
                                                      const uint16_t *__restrict__ vals, PlaceOut out)
{
    __shared__ __attribute__((aligned(16))) uint16_t stage[2 * kSharedWaves][2 * kSharedStage];
    finish_shared_blocks((((int64_t)block0 + blockIdx.x) * kSharedWaves + (threadIdx.x >> 6)) * kSharedPerWave, n_units, V, units, first_vec, win_ptr, blk_ptr, vals, out,
                         stage[threadIdx.x >> 5]);
}

// Other block widths: one block after the other by the whole wavefront.
__global__ void __launch_bounds__(64) k_shared_blocks_any(int block0, int V, int KB, const int4 *__restrict__ units, const int *__restrict__ n_units, const int *__restrict__ first_vec,
                                                          const int32_t *__restrict__ win_ptr, const int *__restrict__ blk_ptr,
                                                          const uint16_t *__restrict__ vals, PlaceOut out)
{
    const int lane = threadIdx.x;
    int my_s = 0, my_kb = 0, my_x = -1;
    const int u = (block0 + blockIdx.x) * kSharedPerWave + lane;
    if (lane < kSharedPerWave && u < *n_units) {
        const int4 un = units[u];
        const SharedBlock sb = shared_block(true, KB, un, first_vec[u], first_vec[max(u - 1, 0)], win_ptr[un.x], win_ptr[un.x + 1], blk_ptr[un.x]);
        my_x = sb.xb; my_s = sb.s; my_kb = sb.kb;
    }
    if (!vals) return;
    for (uint64_t todo = __ballot(my_x >= 0); todo; todo &= todo - 1) {
        const int k = __builtin_ctzll(todo);
        const int xb = __shfl(my_x, k, 64), s = __shfl(my_s, k, 64), kb = __shfl(my_kb, k, 64);
        const uint32_t m = lane < kb ? out.vec_mask[s + lane] : 0u;
        const int32_t base = lane < V ? out.row_base[(int64_t)xb * V + lane] : 0;
        const uint64_t below = (1ull << lane) - 1;
        for (int r = 0; r < V; r++) {
            const bool has = (m >> r) & 1u;
            const int32_t q = __shfl(base, r, 64) + __popcll(__ballot(has) & below);
            if (lane < kb) out.vals_blk[(int64_t)V * s + r * kb + lane] = has ? vals[q] : (uint16_t)0;
        }
    }
}

}  // namespace
