// CSR -> vector-blocked row-window format, entirely on the GPU.
//
// The paper states only that the translation runs as GPU kernels (Section 3.1)
// and what it must produce (Section 3.5); the algorithm below is this
// library's own.  The format's arrays need no sort and no atomics on memory (LDS ones
// only where the order of additions cannot show), so they are deterministic and
// bit-identical to a sequential construction; the work list is sorted, stably:
//
//   1. units  at most 512 stored entries each, one wavefront's work: a few windows, one window, or a range of
//             columns of a hub window (fs_units.h).
//   2. rank   an entry's rank is the number of distinct columns of its unit's window before its own, counted
//             in LDS.  Ranks stay per unit (two bytes per entry); a prefix sum over the units' vector counts gives
//             every unit's first vector, and with it win_ptr.
//   3. place  the same units write vec_col, vec_mask, csr_to_slot, the value array (put together in LDS, so that it
//             is written once, whole), a descriptor per block and, for blocks of 32 vectors, the rows'
//             occupancy and CSR positions and the bitmap-packed copy of the values.
//   4. items  windows longer than one and a half times `chunk` vectors are cut into equal parts of about `chunk`
//             vectors, shorter ones are packed whole into items of about four blocks (counted and then written window by
//             window), and the items are put in launch order.
//
// A small matrix is bound by the number of launches, about 5 us each, and by the two times the host waits,
// for the sizes and at the end.  So a kernel whose results are to be summed leaves the sum of every workgroup, and the next one adds
// up those before its own: no launch only scans (R-MAT of 65 k rows, 0.9 M entries: 17 kernels and 192 us with scans between them,
// ranks by merging and a work list made candidate by candidate, now ten and 149; of 1 M rows, 31 M entries 920 and 752).
#include <algorithm>
#include <cstdlib>

#include "fs_common.h"
#include "fs_scan.h"
#include "fs_sort.h"
#include "fs_units.h"

namespace {

constexpr int kMaxItemBlocks = 32;  // a part of a cut window never has more blocks than this
// ... and no more than this unless the caller asks: with parts launched by column, sixteen-block parts of
// hub windows share more of the dense operand in L2 than thirty-two-block parts do, which outweighs the
// extra partial tiles (cfg 4: 702 us against 720 us per call; eight-block parts 752 us)
constexpr int kDefaultMaxPartBlocks = 16;
constexpr int kPackBlocks = 4;      // packing grain for short windows, in blocks

// Step 4: work items.  Every window owns max(1, ceil(n_w / KB)) block slots, numbered window after
// window.  Items are runs of consecutive slots.  A window with more than 1.5 T blocks is cut into
// round(blocks / T) parts of equal length.  Shorter windows are never cut: candidate boundaries every Ts <= T slots
// snap to the nearest window boundary, so short windows are packed into items of about Ts blocks --
// finer than T, because a block that ends its window (rounding, stores, a narrow operand) costs about
// twice a block inside a long window, and because more, shorter wavefronts keep a CU's memory and LDS
// pipelines busier than few that run in step.
//
// Where items start follows from a window's own slots [lo, hi) and its neighbours', so the list is made window by window, without
// a search (candidate by candidate it took one in the slot table each, 20 k candidates of a 65 k-row R-MAT 8 us, and four launches
// more than a count and a scan of the windows).  Candidate x (a multiple of Ts) in a window that is cut starts the part it lies in;
// in any other it starts an item at lo or, if that is nearer, at hi.  A part has at least Ts slots but for the last, so every part but
// the last holds a candidate, the first one's is the window's first, and an item that begins before the window ends there.
struct WindowCut {
    int plen;   // slots of a part
    int parts;  // items that hold a part of the window; 0: it is not cut
};
__device__ __forceinline__ uint32_t first_candidate(uint32_t lo, int Ts) { return (lo + Ts - 1) / Ts * Ts; }  // at lo or behind it
__device__ __forceinline__ bool is_long(int lo, int hi, int T) { return hi - lo > T + T / 2; }
__device__ __forceinline__ WindowCut window_cut(int lo, int hi, int T, int Ts)
{
    WindowCut c{0, 0};
    const int len = hi - lo;
    if (!is_long(lo, hi, T)) return c;
    // round(len / T) parts of equal length (within one block), so that no part is a short tail -- a part costs an fp32 partial
    // tile whatever its length
    const int parts = (len + T / 2) / T;
    c.plen = (len + parts - 1) / parts;
    c.parts = (int)((uint32_t)(hi - 1) / Ts * Ts - lo) / c.plen + 1;  // up to the last candidate's
    if (c.parts == 1) c.parts = 0;
    return c;
}
// a candidate of window [lo, hi) starts an item at lo (a window of up to one and a half part lengths is kept whole)
__device__ __forceinline__ bool starts_at_lo(int lo, int hi, int T, int Ts)
{
    const uint32_t x = first_candidate(lo, Ts);
    return is_long(lo, hi, T) || (x < (uint32_t)hi && x - lo <= hi - x);
}
// ... at hi
__device__ __forceinline__ bool starts_at_hi(int lo, int hi, int T, int Ts)
{
    const uint32_t x = (uint32_t)(hi - 1) / Ts * Ts;
    return !is_long(lo, hi, T) && x >= (uint32_t)lo && x - lo > hi - x;
}

// T, the blocks per part of a long window, and Ts, the slots between candidates, from the number of block slots NB and those of the longest
// window: enough items to put about 16 wavefronts on each of the 256 CUs, long enough to amortise an item's fixed cost,
// short enough that one item is a small part of the run time.  A caller's own choice of T (t_user > 0) wins; Ts is then as ever, four or T.
// In a small matrix the chain of one item is the time, and shorter items shorten it, but a window cut into parts costs a launch that adds
// them up; so parts are shorter than eight blocks only where some window is cut anyway.  T, Ts = 8, 4 / 4 or 6, 2, us, SpMM with
// 64 and 128 columns and attention with d = 64, N = 128: lognormal graph of 4 k rows 9.2 / 7.2, 10.5 / 8.3, 16.8 / 12.3; R-MAT of 8 k rows, eight entries a
// row, 9.1 / 7.2, 10.5 / 8.2, 17.1 / 11.9, of 16 k, six, 9.8 / 7.6, 11.6 / 9.1, 17.8 / 13.9; stencil of 170^2 points, Ts alone, 6.2 / 5.7, 7.7 / 7.4, 11.0 / 10.3.  Four blocks a
// part for 6 k blocks cost R-MAT of 16 k rows, twelve a row, 3 to 9 %, six for 10 k blocks one of 32 k, eight a row, up to 5.  The conversion does not know
// the width of the products, and wide ones pay for the partial tiles of short parts where hubs hold many of the blocks: R-MAT of 8 k rows, sixteen a row (524 tiles
// of 3.4 k blocks), 128 columns 9.8 / 9.4, 256 10.8 / 11.5, 512 13.4 / 15.2, 1024 20.0 / 22.4; with fewer tiles, R-MAT of 16 k rows, six a row (269 of 4.0 k), 512 15.8 / 15.3.
// From 4 k blocks on three block slots an item pay where windows are long (Ts = 4 / 3: uniform, 20 k rows, twelve a row, three blocks a window, 64 columns
// 7.2 / 6.3, softmax 8.9 / 6.7; lognormal graph of 20 k rows, attention 22.0 / 21.0).  Windows of a block or two may be those of a mesh, whose rows share
// operands with rows a width of the mesh away: items of 32 rows meet them on one XCD where the width is a multiple of 256, and so do
// items of 16, but not of 24 (256^2 points, Ts = 2 / 3 / 4, SpMM with 128 columns 10.5 / 13.6 / 11.2, attention 16.8 / 19.8 / 15.5; with a row of 4000 entries, which
// is cut, 13.7 / 16.6 / 14.9, 21.0 / 24.9 / 21.1).  So there an item has two, where hubs may be the reason that windows are short on
// average (R-MAT of 32 k rows, four a row, 10.5 / 10.5 / 12.6, 15.0 / 14.9 / 19.4), and else four.
struct Grain {
    int T, Ts;
};
__host__ __device__ inline Grain item_grain(int NB, int64_t W, int longest, int t_user, int ts_user)
{
    Grain g;
    if (t_user > 0) {
        g.T = t_user;
        g.Ts = t_user < kPackBlocks ? t_user : kPackBlocks;
    } else {
        const int t = (NB + 4095) / 4096;
        g.T = t < 8 ? 8 : (t > kDefaultMaxPartBlocks ? kDefaultMaxPartBlocks : t);
        if (NB < 4096) g.Ts = 2;
        else if (NB >= 16384) g.Ts = kPackBlocks;
        else if (2 * (int64_t)NB >= 5 * W) g.Ts = 3;
        else g.Ts = longest > g.T + g.T / 2 ? 2 : kPackBlocks;
        if (longest > g.T + g.T / 2 && NB < kShortPartsBelow) g.T = fs_short_part_blocks(NB);
    }
    if (ts_user > 0) g.Ts = ts_user;
    return g;
}

// The window tiles of k_win_ptr: its block slots so far come from its workgroups' sums.  Slots of window w, and of the one before.
__device__ __forceinline__ int window_slots(const int32_t *__restrict__ win_ptr, int64_t w, int KB) { return max(1, (win_ptr[w + 1] - win_ptr[w] + KB - 1) / KB); }

// Per workgroup: items that start in its windows, partial tiles (one per part of a cut window), cut windows.
struct ItemSums {
    int *items, *tiles, *cuts;
};

// Block slots (blk_ptr[W]: their number) and, per workgroup, how many items, partial tiles and cut windows its windows make.
__global__ void __launch_bounds__(kWindowThreads) k_win_slots(const int32_t *__restrict__ win_ptr, int64_t W, int KB, int tiles, const int *__restrict__ slots,
                                                              int t_user, int ts_user, int *__restrict__ blk_ptr, ItemSums sums, int *__restrict__ misc)
{
    if (misc[0] & 1) return;  // malformed row pointers
    const int64_t w0 = (int64_t)blockIdx.x * tiles * kWindowThreads, w1 = min(w0 + (int64_t)tiles * kWindowThreads, W);
    int before[2] = {0, 0};  // the slots of the workgroups before this one, and of all
    for (int k = threadIdx.x; k < (int)gridDim.x; k += kWindowThreads) {
        before[1] += slots[k];
        if (k < (int)blockIdx.x) before[0] = before[1];
    }
    block_sum<kWindowThreads>(before);
    int ahead = before[0];
    const int NB = before[1];
    const Grain grain = item_grain(NB, W, misc[2], t_user, ts_user);
    const int T = grain.T, Ts = grain.Ts;
    int n[3] = {0, 0, 0};  // items, partial tiles, cut windows
    for (int64_t wt = w0; wt < w1; wt += kWindowThreads) {
        const int64_t w = wt + threadIdx.x;
        const int mine = w < w1 ? window_slots(win_ptr, w, KB) : 0;
        const int prev = w > 0 && w < w1 ? window_slots(win_ptr, w - 1, KB) : 0;
        int here;
        const int lo = ahead + block_exclusive_scan<kWindowThreads>(mine, &here), hi = lo + mine;
        ahead += here;
        if (w >= w1) continue;
        blk_ptr[w] = lo;
        const WindowCut c = window_cut(lo, hi, T, Ts);
        n[0] += (starts_at_lo(lo, hi, T, Ts) || (w > 0 && starts_at_hi(lo - prev, lo, T, Ts)) ? 1 : 0) + max(c.parts - 1, 0);
        if (w == W - 1) {
            blk_ptr[W] = hi;
            n[0] += starts_at_hi(lo, hi, T, Ts) ? 1 : 0;  // a record of no blocks, the last
        }
        n[1] += c.parts;
        n[2] += c.parts > 0 ? 1 : 0;
    }
    block_sum<kWindowThreads>(n);
    if (threadIdx.x == 0) {
        sums.items[blockIdx.x] = n[0];
        sums.tiles[blockIdx.x] = n[1];
        sums.cuts[blockIdx.x] = n[2];
        if (blockIdx.x == 0) misc[4] = NB;
        // counts: the same whatever the order of the additions (one atomic operation for two of them, they are what the workgroups wait for)
        atomicAdd(reinterpret_cast<unsigned long long *>(misc + 6), (unsigned long long)(uint32_t)n[1] << 32 | (uint32_t)n[0]);
        if (n[2]) atomicAdd(&misc[5], n[2]);
    }
}

// Launch order of the work list.  Parts of cut windows come first, ordered by the column of their first
// vector: a hub window references a broad, mostly cold set of columns in ascending order, so parts that
// start at the same column sweep the same rows of the dense operand and, run side by side, share them in
// L2 instead of fetching them once per window.  Whole windows follow, the costliest items first (one unit
// per block and one more per block that ends its window: rounding, stores and a narrow operand make such
// a block about twice as dear), so that the wavefronts still running when the launch drains are short
// ones and the short windows, whose vectors sit on the hot columns, are not mixed with the cold sweep of
// the hubs.  Measured against the work list's own order: cfg 2 k_spmm 24.0 -> 21.5 us, cfg 4 (four-row
// windows) 938 -> 827 us with the cost order alone.  The 24-bit key sorts ascending; equal keys keep the
// work list's order (the sort is stable).
// The item records {first block slot, blocks, first partial slot, first vector} with their keys, the table of cut windows and, for
// every partial slot, its window's slot range, again window by window.  An item that starts at a window's first slot, or with its last
// part, ends where the next item of the windows behind it starts: at the first candidate from there on, which lies less than Ts windows
// away.  With Ts <= T <= 32 no item exceeds the 64 block descriptors a wavefront holds: parts have at most 1.25 T + 1 blocks, whole
// windows 1.5 T, and packing adds less than 3 Ts.  The parts of cut windows are dealt to the threads one by one, and in a
// long list to the threads of several workgroups, because the hubs of a graph lie side by side (R-MAT of 1 M rows, 60 k parts: written by
// the wavefront of their window 51 us, by one workgroup 30, by four 23).
__device__ __forceinline__ void fill_items(int group, int share, int shares, const int *__restrict__ blk_ptr, int64_t W, int tiles, Grain grain, ItemSums sums,
                                                   const int32_t *__restrict__ win_ptr, int KB, const int32_t *__restrict__ vec_col,
                                                   int64_t nvec, int64_t K, int n_items, int4 *__restrict__ items, int32_t *__restrict__ key,
                                                   int4 *__restrict__ split_windows, int2 *__restrict__ slot_range)
{
    // of the tile's cut windows, in order: parts before them, {first slot, slots a part, end of the last item, first vector}, {first item, parts}
    __shared__ int part_of[kWindowThreads];
    __shared__ int4 cut_at[kWindowThreads];
    __shared__ int2 cut_items[kWindowThreads];
    const int64_t w0 = (int64_t)group * tiles * kWindowThreads, w1 = min(w0 + (int64_t)tiles * kWindowThreads, W);
    const int NB = blk_ptr[W], T = grain.T, Ts = grain.Ts;
    int ahead[3] = {0, 0, 0};  // items, partial tiles, cut windows of the workgroups before this one
    for (int k = threadIdx.x; k < group; k += kWindowThreads) {
        ahead[0] += sums.items[k];
        ahead[1] += sums.tiles[k];
        ahead[2] += sums.cuts[k];
    }
    block_sum<kWindowThreads>(ahead);
    const bool parts_only = share > 0;
    if (!parts_only && group == 0 && threadIdx.x < 64 && n_items + (int)threadIdx.x < (n_items + 63) / 64 * 64)
        key[n_items + threadIdx.x] = INT32_MAX;  // (k_item_rank reads 64 keys at a time)
    for (int64_t wt = w0; wt < w1; wt += kWindowThreads) {
        const int64_t w = wt + threadIdx.x;
        const bool live = w < w1;
        const int lo = live ? blk_ptr[w] : 0, hi = live ? blk_ptr[w + 1] : 0, lo_prev = live && w > 0 ? blk_ptr[w - 1] : 0;
        const int q = live ? win_ptr[w] : 0;
        const WindowCut c = live ? window_cut(lo, hi, T, Ts) : WindowCut{0, 0};
        const bool begins = live && (starts_at_lo(lo, hi, T, Ts) || (w > 0 && starts_at_hi(lo_prev, lo, T, Ts)));
        const bool nothing = live && w == W - 1 && starts_at_hi(lo, hi, T, Ts);  // a record of no blocks, the last
        int n_i, n_t, n_c;
        const int item = ahead[0] + block_exclusive_scan<kWindowThreads>((begins ? 1 : 0) + max(c.parts - 1, 0) + (nothing ? 1 : 0), &n_i);
        const int part = block_exclusive_scan<kWindowThreads>(c.parts, &n_t), cut = block_exclusive_scan<kWindowThreads>(c.parts > 0 ? 1 : 0, &n_c);
        // where the item ends that the window's first slot or last part begins, and the windows that end in it
        int end = hi, ends = 1;
        if ((c.parts > 0 || (begins && !parts_only)) && !starts_at_hi(lo, hi, T, Ts)) {
            const uint32_t x = first_candidate(hi, Ts);  // the next candidate; it lies in the first window that ends behind it
            end = NB;
            int64_t v = w + 1;
            int lo_v = hi;
            for (; v < W; v++) {
                const int hi_v = blk_ptr[v + 1];
                if ((uint32_t)hi_v > x) {
                    end = lo_v;
                    if (!starts_at_lo(lo_v, hi_v, T, Ts)) { end = hi_v; v++; }
                    break;
                }
                lo_v = hi_v;
            }
            ends = (int)(v - w);
        }
        if (nothing && !parts_only) {
            items[item + (begins ? 1 : 0)] = make_int4(0, 0, 0, 0);
            key[item + (begins ? 1 : 0)] = 0x00FFFFFF;  // empty record: last
        }
        if (begins && c.parts == 0 && !parts_only) {
            items[item] = make_int4(lo, end - lo, ahead[1] + part, q);
            key[item] = (1 + 128 - min(end - lo + ends, 128)) << 16;  // blocks, and blocks that end a window
        }
        if (c.parts > 0) {
            if (!parts_only) split_windows[ahead[2] + cut] = make_int4((int)w, ahead[1] + part, c.parts, 0);
            part_of[cut] = part;
            cut_at[cut] = make_int4(lo, c.plen, end, q);
            cut_items[cut] = make_int2(item, c.parts);
        }
        __syncthreads();
        for (int f = share * kWindowThreads + threadIdx.x; f < n_t; f += shares * kWindowThreads) {
            int k = 0;  // the cut window of part f: the last that begins with it or before
            for (int h = kWindowThreads >> 1; h > 0; h >>= 1) k += k + h < n_c && part_of[k + h] <= f ? h : 0;
            const int4 at = cut_at[k];
            const int2 its = cut_items[k];
            const int m = f - part_of[k], s = at.x + m * at.y, v = at.w + m * at.y * KB, slot = ahead[1] + f;
            const int32_t column = nvec > 0 ? vec_col[min((int64_t)v, nvec - 1)] : 0;
            items[its.x + m] = make_int4(s, (m + 1 < its.y ? s + at.y : at.z) - s, slot, v);
            key[its.x + m] = (int32_t)(((int64_t)column << 16) / max(K, (int64_t)1));  // column of the first vector, 16 bits
            slot_range[slot] = make_int2(slot - m, its.y);
        }
        __syncthreads();
        ahead[0] += n_i;
        ahead[1] += n_t;
        ahead[2] += n_c;
    }
}

// What is left when the units are placed: the work list, by the first groups * shares workgroups, and, where they are few, the blocks that
// pieces of hub windows share, by the others: a launch less where launches are the time (R-MAT of 65 k rows 9 and 5 us, now 9).
struct ItemFill {
    int groups, shares, tiles, n_items;
    Grain grain;
    ItemSums sums;
    int4 *items;
    int32_t *key;
    int4 *split_windows;
    int2 *slot_range;
};
__global__ void __launch_bounds__(kWindowThreads) __attribute__((amdgpu_waves_per_eu(4))) k_finish(ItemFill fill, const int *__restrict__ blk_ptr, int64_t W, const int32_t *__restrict__ win_ptr, int KB, int64_t nvec, int64_t K,
                                                           int V, const int4 *__restrict__ units, int n_units, const int *__restrict__ first_vec,
                                                           const uint16_t *__restrict__ vals, PlaceOut out)
{
    const int first = fill.groups * fill.shares;
    if ((int)blockIdx.x < first) {
        fill_items(blockIdx.x % fill.groups, blockIdx.x / fill.groups, fill.shares, blk_ptr, W, fill.tiles, fill.grain, fill.sums, win_ptr, KB, out.vec_col, nvec, K,
                   fill.n_items, fill.items, fill.key, fill.split_windows, fill.slot_range);
        return;
    }
    constexpr int kWaves = kWindowThreads / 64;
    __shared__ __attribute__((aligned(16))) uint16_t stage[kWaves * 2][2 * kSharedStage];
    finish_shared_blocks((int64_t)(((int)blockIdx.x - first) * kWaves + (threadIdx.x >> 6)) * kSharedPerWave, n_units, V, units, first_vec, win_ptr, blk_ptr, vals, out, stage[threadIdx.x >> 5]);
}

// The work list in launch order: by_cost[t] = items[order[t]], so that a wavefront finds its item with one load.
__global__ void k_item_permute(const int4 *__restrict__ items, const int32_t *__restrict__ order, int n_items,
                               int4 *__restrict__ by_cost)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n_items) by_cost[t] = items[order[t]];
}

__device__ __forceinline__ void count_if_less(int &n, int32_t key, int32_t x)  // n += key < x
{
    asm("v_cmp_lt_i32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc" : "+v"(n) : "v"(key), "v"(x) : "vcc");
}
// The same for a short list, in one launch: an item's place is the number of keys before its own.  A workgroup takes 32
// items; each half of its sixteen wavefronts compares them with its share of the keys, 64 at a time by way of LDS, two
// instructions a comparison.  keys: padded to a multiple of 64 with keys larger than all.  5226 items: 22 us by one
// workgroup that sorted them in three digit passes, now 8; from about 24 k items on the radix passes are the shorter way.
constexpr int kRankItemsMax = 16384, kRankWaves = 16, kRankItems = 32;
constexpr int kKeyDigitBits = 8, kKeyDigits = 1 << kKeyDigitBits;  // of the radix passes
__global__ void __launch_bounds__(64 * kRankWaves) k_item_rank(const int32_t *__restrict__ keys, int n, const int4 *__restrict__ items,
                                                               int32_t *__restrict__ order, int4 *__restrict__ by_cost)
{
    __shared__ __attribute__((aligned(16))) int32_t share[kRankWaves][2][64 + 4];  // the halves' keys, in different banks
    __shared__ int part[2 * kRankWaves][kRankItems];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, half = lane >> 5;
    const int i = blockIdx.x * kRankItems + (lane & 31), i0 = i & ~63;  // i0: the group of keys its own is in
    const int32_t mine = keys[i];
    const int groups = (n + 63) / 64;
    int before = 0;
    for (int g0 = 2 * w; g0 < groups; g0 += 2 * kRankWaves) {
        share[w][0][lane] = keys[g0 * 64 + lane];
        share[w][1][lane] = g0 + 1 < groups ? keys[g0 * 64 + 64 + lane] : INT32_MAX;
        FS_WAVE_SYNC();
        const int j0 = (g0 + half) * 64;
        const int32_t bound = j0 < i0 ? mine + 1 : mine;  // of earlier items, equal keys come first
        const int4 *k4 = reinterpret_cast<const int4 *>(share[w][half]);
        if (j0 != i0) {
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const int4 k = k4[q];
                count_if_less(before, k.x, bound);
                count_if_less(before, k.y, bound);
                count_if_less(before, k.z, bound);
                count_if_less(before, k.w, bound);
            }
        } else {
            for (int j = 0; j < 64; j++) {
                const int32_t k = share[w][half][j];
                before += k < mine || (k == mine && j0 + j < i) ? 1 : 0;
            }
        }
        FS_WAVE_SYNC();
    }
    part[2 * w + half][lane & 31] = before;
    __syncthreads();
    if (threadIdx.x >= kRankItems || i >= n) return;
    int at = 0;
#pragma unroll
    for (int k = 0; k < 2 * kRankWaves; k++) at += part[k][lane];
    order[at] = i;
    by_cost[at] = items[i];
}

// CSR position of the first stored entry of window row r that lies in block slot x or later:
// row_base[x * V + r] = first position in row w*V + r whose column is >= the column of the block's first
// vector.  With the block's occupancy bits this gives the CSR position of every entry of the block, which
// lets a kernel that works block by block write its results in CSR order.  (Blocks of 32 vectors have it from
// k_unit_place; this is for the other widths.)
__global__ void k_block_row_base(CsrView a, int V, const int4 *__restrict__ blk_desc, int NB,
                                 const int32_t *__restrict__ vec_col, int64_t nvec, int32_t *__restrict__ row_base)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)NB * V) return;
    const int x = (int)(t / V), r = (int)(t - (int64_t)x * V);
    const int4 d = blk_desc[x];
    const int64_t row = (int64_t)d.z * V + r;
    int32_t lo = 0, hi = 0;
    if (row < a.M) row_range(a, row, lo, hi);
    if ((d.y & 255) > 0 && nvec > 0) {
        const int32_t c = vec_col[min((int64_t)d.x, nvec - 1)];
        while (lo < hi) {
            const int32_t mid = lo + ((hi - lo) >> 1);
            if (a.colidx[mid] < c) lo = mid + 1; else hi = mid;
        }
    }
    row_base[t] = lo;
}

template <typename T>
__global__ void k_blk_to_csr(const int32_t *__restrict__ csr_to_slot, const T *__restrict__ blk, T *__restrict__ out, int64_t nnz)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nnz) out[p] = blk[csr_to_slot[p]];
}

// 16-byte pieces of zeros (the blocked value array is 16-byte aligned and padded to 16 bytes by its owner)
__global__ void k_zero16(fs_u4 *__restrict__ dst, int64_t n16)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = fs_u4{0u, 0u, 0u, 0u};
}

template <typename T>
__global__ void k_zero_tail(T *__restrict__ dst, int64_t from, int64_t to)
{
    int64_t i = from + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < to) dst[i] = (T)0;
}

template <typename T>
__global__ void k_csr_to_blk(const int32_t *__restrict__ csr_to_slot, const T *__restrict__ vals, T *__restrict__ blk, int64_t nnz)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nnz) blk[csr_to_slot[p]] = vals[p];
}

// Values in CSR order -> the value array, blocks of 32 vectors.  Lane (block b, row j, group g) of a round takes the entries of row
// j among vectors 8g .. 8g+7, which follow each other in CSR order, from one 16-byte load, and spreads them by the row's
// occupancy; the tiles of a wavefront's blocks follow each other in the array, so they are put together in LDS
// and leave in one contiguous run.  Each element is written once, zeros included: 59 MB for 5.3 M entries in four-row
// windows, where clearing the array and scattering single elements through csr_to_slot moved 116 MB in three launches: 24 us on
// arrays the last-level cache holds, now 14; among the kernels of a training step 31, now 19.
template <int V>
__global__ void __launch_bounds__(256) k_csr_to_tiles(const int4 *__restrict__ blk_desc, int n_blocks, const uint32_t *__restrict__ row_bits,
                                                      const int32_t *__restrict__ row_base, const uint16_t *__restrict__ vals, int nnz, uint16_t *__restrict__ out)
{
    constexpr int ROUNDS = 2, PER = 16 / V;  // blocks per round
    constexpr int PIECE = V % 8 == 0 ? 8 : 4;   // elements that share alignment with every tile
    __shared__ __attribute__((aligned(16))) uint16_t tiles[4][ROUNDS * 512];
    __shared__ uint2 sels[4][16];
    const int lane = threadIdx.x & 63;
    uint2 *sel = sels[threadIdx.x >> 6];
    fs_expand_table(sel, lane);
    uint16_t *tile = tiles[threadIdx.x >> 6];
    const int g = lane & 3, j = (lane >> 2) % V, b = (lane >> 2) / V;
    const int x0 = (int)((blockIdx.x * 4 + (threadIdx.x >> 6)) * (PER * ROUNDS));
    if (x0 >= n_blocks) return;  // no block-wide barrier is used below
    int4 d[ROUNDS];
    uint32_t bits[ROUNDS], m8[ROUNDS];
    int pos[ROUNDS];
    fs_u4 raw[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        const int x = min(x0 + r * PER + b, n_blocks - 1);
        d[r] = blk_desc[x];
        bits[r] = row_bits[(int64_t)x * V + j];
        pos[r] = row_base[(int64_t)x * V + j];
        if (x0 + r * PER + b >= n_blocks) d[r].y = 0;
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        m8[r] = bits[r] >> (8 * g) & 0xFFu;
        pos[r] += __popc(bits[r] & ((1u << (8 * g)) - 1u));
        const uint16_t *src = vals + max(min(pos[r], nnz - 8), 0);
        if (nnz >= 8) raw[r] = *reinterpret_cast<const fs_u4_unaligned *>(src);
    }
    int end = 0;
    const int s0 = __builtin_amdgcn_readfirstlane(d[0].x);
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        const int kb = d[r].y & 255;
        if (pos[r] + 8 > nnz) {  // the matrix' last entries
            fs_frag o;
            o.u = fs_u4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int k = 0; k < 8; k++) o.e[k] = pos[r] + k < nnz ? vals[pos[r] + k] : (uint16_t)0;
            raw[r] = o.u;
        }
        fs_frag o;
        o.u = fs_expand8(raw[r], m8[r], sel);
        uint16_t *at = tile + V * (d[r].x - s0) + j * kb + 8 * g;
        if (kb == 32) {
            if constexpr (PIECE == 8) {
                *reinterpret_cast<fs_u4 *>(at) = o.u;
            } else {
                *reinterpret_cast<uint2 *>(at) = make_uint2(o.u.x, o.u.y);
                *reinterpret_cast<uint2 *>(at + 4) = make_uint2(o.u.z, o.u.w);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (8 * g + k < kb) at[k] = o.e[k];
        }
        if (kb > 0) end = d[r].x + kb - s0;
    }
    for (int h = 4 * V; h < 64; h <<= 1) end = max(end, __shfl_xor(end, h, 64));  // of the wavefront's last block
    FS_WAVE_SYNC();
    uint16_t *dst = out + (int64_t)V * s0;
    for (int i = lane * PIECE; i < V * end; i += 64 * PIECE) {
        if constexpr (PIECE == 8) *reinterpret_cast<fs_u4 *>(dst + i) = *reinterpret_cast<const fs_u4 *>(tile + i);
        else *reinterpret_cast<uint2 *>(dst + i) = *reinterpret_cast<const uint2 *>(tile + i);
    }
}

// Stored entries per block slot (the sum of the occupancy bits of its vectors): half a wavefront per slot,
// one lane per vector.  The same pass writes every vector's occupancy mask narrowed to one byte (m8, for
// V <= 8) or two (m16), the form the packed-value kernels read.
__global__ void __launch_bounds__(256) k_block_nnz(const int4 *__restrict__ blk_desc, int64_t n_blocks,
                                                   const uint32_t *__restrict__ vec_mask, int32_t *__restrict__ cnt,
                                                   uint8_t *__restrict__ m8, uint16_t *__restrict__ m16)
{
    const int lane = threadIdx.x & 63, c = lane & 31;
    const int64_t b = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 2 + (lane >> 5);
    int n = 0;
    if (b < n_blocks) {
        const int4 d = blk_desc[b];
        if (c < (d.y & 255)) {
            const uint32_t m = vec_mask[d.x + c];
            n = __popc(m);
            if (m8) m8[d.x + c] = (uint8_t)m; else m16[d.x + c] = (uint16_t)m;
        }
    }
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) n += __shfl_xor(n, o, 64);  // the 32 lanes of the half
    if (c == 0 && b < n_blocks) cnt[b] = n;
}

// Half a wavefront per block slot (at most 32 vectors): the stored values of the V x kb tile, row after
// row, go to consecutive positions from blk_ofs[slot] on.  Lane c < kb owns vector c and reads its column
// of the tile first, all rows at once; its position inside row r is the number of lower lanes of its half
// that also store row r.
__global__ void __launch_bounds__(256) k_pack(const int4 *__restrict__ blk_desc, int64_t n_blocks, int V,
                                              const uint32_t *__restrict__ vec_mask, const uint16_t *__restrict__ vals_blk,
                                              const int32_t *__restrict__ blk_ofs, uint16_t *__restrict__ packed)
{
    constexpr int kMaxV = 16;
    const int lane = threadIdx.x & 63, c = lane & 31, half = lane >> 5;
    const int64_t b = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 2 + half;
    int s = 0, kb = 0;
    if (b < n_blocks) {
        const int4 d = blk_desc[b];
        s = d.x;
        kb = d.y & 255;
    }
    const bool mine = c < kb;
    const uint32_t msk = mine ? vec_mask[s + c] : 0u;
    int pos = mine ? blk_ofs[b] : 0;
    const uint16_t *tile = vals_blk + (int64_t)V * s;
    uint16_t v[kMaxV];
#pragma unroll
    for (int r = 0; r < kMaxV; r++) v[r] = (r < V && mine) ? tile[r * kb + c] : (uint16_t)0;
    const uint32_t below = (1u << c) - 1u;
#pragma unroll
    for (int r = 0; r < kMaxV; r++) {
        if (r >= V) break;
        const bool has = (msk >> r) & 1u;
        const uint64_t both = __ballot(has);
        const uint32_t row = (uint32_t)(half ? both >> 32 : both);
        if (has) packed[pos + __popc(row & below)] = v[r];
        pos += __popc(row);
    }
}

inline unsigned grid_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

// Scratch layout (ints): [ranks: nnz 16-bit][scan tmp][err + totals: 64][units, 4 each][where they start in their rows, V each][their vector counts + 1]
// [their first vectors + 1][windows' places in them, 2 each][blk_ptr: W+1][windows to cut again: W+1][sums per workgroup, five times]
// [keys of the work list, twice][its order][digit counts of its sort]
struct ScratchPlan {
    size_t info, tmp, misc, units, pieces, count, first, win_at, blk, redo, sums, key0, key1, order, hist, total_ints;
};
size_t items_bound(int64_t W, int64_t nnz, int KB) { return (size_t)(W + nnz / KB + 2); }
ScratchPlan plan_scratch(int64_t nnz, int64_t W, int V, int KB)
{
    ScratchPlan s;
    const size_t ib = items_bound(W, nnz, KB), ub = (size_t)units_bound(W, nnz);
    size_t o = 0;
    s.info = o; o += fs_align_up(((size_t)nnz + 1) / 2, 64);
    s.tmp = o; o += scan_tmp_ints(std::max<int64_t>(std::max<int64_t>(nnz, W), (int64_t)ib));
    s.misc = o; o += 64;
    s.units = o; o += fs_align_up(4 * ub, 64);
    s.pieces = o; o += fs_align_up(ub * V, 64);
    s.count = o; o += fs_align_up(ub + 1, 64);
    s.first = o; o += fs_align_up(ub + 1, 64);
    s.win_at = o; o += fs_align_up(2 * (size_t)W, 64);
    s.blk = o; o += fs_align_up((size_t)W + 1, 64);
    s.redo = o; o += fs_align_up((size_t)W + 1, 64);
    s.sums = o; o += 5 * kScanDirect;
    s.key0 = o; o += fs_align_up(ib, 64);
    s.key1 = o; o += fs_align_up(ib, 64);
    s.order = o; o += fs_align_up(ib, 64);
    s.hist = o; o += fs_align_up((size_t)kKeyDigits * sort_groups_bound((int64_t)ib) + 1, 64);  // digit counts of the work-list sort
    s.total_ints = std::max(o, (size_t)nnz);  // (never less than the four bytes per entry of earlier layouts)
    return s;
}

// Window height when the caller leaves the choice to the library: eight rows, which are best or within a few
// per cent of best on every workload measured -- except on large fabric-bound matrices whose rows share
// almost no columns inside an eight-row window: there a taller window saves no vectors and a four-row
// window halves the value array for everything that reads it unpacked (cfg 5: SpMM on SDDMM scores 381 us
// against 401 us; cfg 4, whose windows do share columns, 779 us against 750 us the other way).  So for a
// matrix that qualifies for packed values the conversion counts the vectors at eight rows first and starts
// over with four when fewer than one stored entry in twenty shares its vector with another.
int32_t default_window_rows(int64_t, int64_t) { return 8; }
bool prefers_four_rows(int64_t nnz, int64_t nvec_at_eight) { return nvec_at_eight * 20 > nnz * 19; }

// Large matrices with long rows are bound by the memory fabric: for them the conversion also packs the
// values (only the stored ones, see fs_pack_values) and fs_spmm reads those.  On small or short-row
// matrices decoding costs more than the traffic it saves (cfg 2 +9 %, cfg 3 +4 %).
bool wants_packed_values(int64_t M, int64_t nnz, int32_t V, int32_t KB)
{
    return nnz >= ((int64_t)1 << 22) && nnz >= 12 * M && KB == 32 && V <= 16;
}

bool params_ok(int64_t M, int64_t nnz, int32_t V, int32_t KB)
{
    return M >= 0 && nnz >= 0 && V >= 1 && V <= 32 && KB >= 1 && KB <= 64;
}

}  // namespace

extern "C" fs_status fs_format_bytes(int64_t M, int64_t nnz, int32_t V, int32_t KB, fs_dtype dtype,
                                     size_t *arena_bytes, size_t *scratch_bytes)
{
    if (KB == 0) KB = 32;
    if (V == 0) {  // the library may settle on eight or on four rows: room for either
        size_t a8 = 0, s8 = 0, a4 = 0, s4 = 0;
        fs_status st = fs_format_bytes(M, nnz, 8, KB, dtype, &a8, &s8);
        if (st != FS_OK) return st;
        if ((st = fs_format_bytes(M, nnz, 4, KB, dtype, &a4, &s4)) != FS_OK) return st;
        if (arena_bytes) *arena_bytes = std::max(a8, a4);
        if (scratch_bytes) *scratch_bytes = std::max(s8, s4);
        return FS_OK;
    }
    if (!params_ok(M, nnz, V, KB) || (dtype != FS_F16 && dtype != FS_BF16)) return FS_ERR_INVALID_ARG;
    if (nnz >= (int64_t)1 << 31 || M >= (int64_t)1 << 31 || (int64_t)V * nnz >= (int64_t)1 << 31) return FS_ERR_TOO_LARGE;
    const int64_t W = (M + V - 1) / V;
    if (arena_bytes) {
        size_t a = 0;
        a += fs_align_up((size_t)(W + 1) * 4, 256);            // win_ptr
        a += 3 * fs_align_up((size_t)nnz * 4, 256);            // vec_col, vec_mask, csr_to_slot
        a += fs_align_up((size_t)V * nnz * 2, 256) + 256;      // vals_blk (+ slack so a 16-byte read of the tail stays inside)
        a += 3 * fs_align_up(items_bound(W, nnz, KB) * 16, 256);  // blk_desc, items, split_windows
        a += fs_align_up(items_bound(W, nnz, KB) * 4, 256);       // item_order
        a += 2 * fs_align_up(items_bound(W, nnz, KB) * V * 4, 256);  // blk_row_base, blk_row_bits
        a += fs_align_up(items_bound(W, nnz, KB) * 16, 256);      // items_by_cost
        a += fs_align_up(items_bound(W, nnz, KB) * 16, 256);      // slot_range (an item has at most two partial tiles)
        if (wants_packed_values(M, nnz, V, KB)) {  // the packed copy of the values (bounds: nvec <= nnz, blocks <= items_bound)
            fs_format b{};
            b.n_blocks = (int64_t)items_bound(W, nnz, KB); b.nvec = nnz; b.nnz = nnz; b.V = V;
            a += fs_packed_plan(&b).total + 256;
        }
        *arena_bytes = a;
    }
    if (scratch_bytes) *scratch_bytes = plan_scratch(nnz, W, V, KB).total_ints * 4;
    return FS_OK;
}

extern "C" fs_status fs_convert(int64_t M, int64_t K, int64_t nnz, const int32_t *d_rowptr, const int32_t *d_colidx,
                                const void *d_vals, fs_dtype dtype, int32_t V, int32_t KB, int32_t chunk,
                                void *d_arena, size_t arena_bytes, void *d_scratch, size_t scratch_bytes,
                                void *stream, fs_format *out)
{
    const bool library_picks_rows = V == 0;
    if (V == 0) V = default_window_rows(M, nnz);
    if (KB == 0) KB = 32;
    if (!out || !d_rowptr || !d_arena || !d_scratch || K < 0 || (nnz > 0 && (!d_colidx || M == 0))) return FS_ERR_INVALID_ARG;
    size_t need_arena = 0, need_scratch = 0;
    fs_status st = fs_format_bytes(M, nnz, library_picks_rows ? 0 : V, KB, dtype, &need_arena, &need_scratch);
    if (st != FS_OK) return st;
    if (chunk < 0 || (chunk > 0 && (chunk % KB != 0 || chunk / KB > kMaxItemBlocks))) return FS_ERR_INVALID_ARG;
    if (((uintptr_t)d_arena | (uintptr_t)d_scratch) & 255) return FS_ERR_INVALID_ARG;
    if (arena_bytes < need_arena || scratch_bytes < need_scratch) return FS_ERR_BUFFER_TOO_SMALL;

    hipStream_t s = (hipStream_t)stream;
    const int64_t W = (M + V - 1) / V;
    const ScratchPlan sp = plan_scratch(nnz, W, V, KB);
    int *scr = (int *)d_scratch;
    int *misc = scr + sp.misc, *tmp = scr + sp.tmp;
    int *blk_ptr = scr + sp.blk, *redo = scr + sp.redo;
    int32_t *key0 = scr + sp.key0, *key1 = scr + sp.key1, *order = scr + sp.order;
    uint16_t *info = (uint16_t *)(scr + sp.info);
    int4 *units = (int4 *)(scr + sp.units);
    int *pieces = scr + sp.pieces, *count = scr + sp.count, *first_vec = scr + sp.first;
    int2 *win_at = (int2 *)(scr + sp.win_at);
    int *sums = scr + sp.sums;  // per workgroup: units, block slots, items, partial tiles, cut windows
    const ItemSums item_sums{sums + 2 * kScanDirect, sums + 3 * kScanDirect, sums + 4 * kScanDirect};
    char *arena = (char *)d_arena;
    int32_t *win_ptr = (int32_t *)arena;
    CsrView a{d_rowptr, d_colidx, M, (int32_t)nnz};

    // misc: [0] CSR error flags, [1] vectors, [2] block slots of the longest window, [4] block slots, [5] cut windows, [6] items, [7] partial tiles (and items that hold a
    // part of a cut window: one each), [8] units -- what the host reads, in one copy
    FS_HIP(hipMemsetAsync(misc, 0, 64 * sizeof(int), s));
    const UnitPlan up = unit_plan(nnz, V);
    const int64_t max_units = units_bound(up, W, nnz);
    int *n_units = misc + 8;
    // workgroups whose sums the next kernel adds up: at most kScanDirect, so each takes as many tiles of windows as that needs
    auto tiles_for = [&](int64_t per_tile) -> int { return (int)std::max<int64_t>((W + per_tile * kScanDirect - 1) / (per_tile * kScanDirect), 1); };
    auto groups_for = [&](int64_t per_tile, int tiles) -> unsigned { return grid_for(std::max<int64_t>(W, 1), (int)(per_tile * tiles)); };
    const int unit_tiles = tiles_for(kCountGroups * up.group), tiles = tiles_for(kWindowThreads);
    const unsigned unit_grid = groups_for(kCountGroups * up.group, unit_tiles), win_grid = groups_for(kWindowThreads, tiles);
    k_units_count<<<unit_grid, kCountThreads, 0, s>>>(a, up, W, unit_tiles, sums, misc);
    FS_LAUNCH_CHECK();
    const int *count_sums = nullptr;
    bool scanned = false;
    if (W > 0) {
        k_units_fill<<<unit_grid, kCountThreads, 0, s>>>(a, up, W, unit_tiles, sums, units, n_units, redo, misc);
        FS_LAUNCH_CHECK();
        if (nnz > kUnitEntries) {
            st = launch_units(V <= 8 ? (max_units + 6) / 7 : V <= 16 ? (max_units + 2) / 3 : max_units, [&](int first, unsigned grid) {
                if (V <= 8) k_pieces<8><<<grid, 64, 0, s>>>(first, a, up, units, n_units, pieces, redo, misc);
                else if (V <= 16) k_pieces<16><<<grid, 64, 0, s>>>(first, a, up, units, n_units, pieces, redo, misc);
                else k_pieces<32><<<grid, 64, 0, s>>>(first, a, up, units, n_units, pieces, redo, misc);
            });
            if (st != FS_OK) return st;
            st = launch_units((max_units + kExactPerWave - 1) / kExactPerWave, [&](int first, unsigned grid) {
                if (V <= 8) k_pieces_exact<8><<<grid, 64, 0, s>>>(first, a, up, units, n_units, pieces, redo, misc);
                else if (V <= 16) k_pieces_exact<16><<<grid, 64, 0, s>>>(first, a, up, units, n_units, pieces, redo, misc);
                else k_pieces_exact<32><<<grid, 64, 0, s>>>(first, a, up, units, n_units, pieces, redo, misc);
            });
            if (st != FS_OK) return st;
        }
        k_unit_rank<<<(unsigned)std::min<int64_t>(max_units, kRankGrid), 64, 0, s>>>(a, up, K, units, n_units, pieces, info, count, win_at, misc);
        FS_LAUNCH_CHECK();
        // Up to 16 k units every workgroup of k_win_ptr adds up the counts before its own itself, 64 KB at most; more are summed
        // beforehand, kScanTile at a time.
        if (max_units > 16384) {
            const int64_t n_sums = (max_units + kScanTile - 1) / kScanTile;
            k_scan_reduce<<<(unsigned)n_sums, kScanThreads, 0, s>>>(count, max_units, tmp);
            FS_LAUNCH_CHECK();
            scanned = n_sums > kScanDirect;
            if (scanned && (st = scan_exclusive(tmp, n_sums, tmp + fs_align_up((size_t)n_sums + 1, 64), s)) != FS_OK) return st;
            count_sums = tmp;
        }
    }
    k_win_ptr<<<win_grid, kWindowThreads, 0, s>>>(win_at, count, count_sums, scanned, n_units, W, KB, tiles, first_vec, win_ptr, sums + kScanDirect, misc);
    FS_LAUNCH_CHECK();

    // Work items (step 4), up to their count: their grain follows from the number of block slots and the longest window, which the
    // kernels read from the device.
    const int t_user = chunk > 0 ? chunk / KB : 0;
    int ts_user = 0;
#ifdef FS_TUNING_ENV
    if (const char *e = getenv("FS_PACK_BLOCKS")) ts_user = std::max(std::min(atoi(e), t_user > 0 ? t_user : 4), 1);
#endif
    if (W > 0) {
        k_win_slots<<<win_grid, kWindowThreads, 0, s>>>(win_ptr, W, KB, tiles, sums + kScanDirect, t_user, ts_user, blk_ptr, item_sums, misc);
        FS_LAUNCH_CHECK();
    }

    int h_misc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    FS_HIP(hipMemcpyAsync(h_misc, misc, sizeof(h_misc), hipMemcpyDeviceToHost, s));
    FS_HIP(hipStreamSynchronize(s));
    if (h_misc[0]) return FS_ERR_INVALID_CSR;
    const int64_t nvec = h_misc[1];
    const int NB = h_misc[4];  // block slots in total
    const int units_made = h_misc[8];
    if (library_picks_rows && V == 8 && wants_packed_values(M, nnz, 4, KB) && prefers_four_rows(nnz, nvec))
        return fs_convert(M, K, nnz, d_rowptr, d_colidx, d_vals, dtype, 4, KB, chunk, d_arena, arena_bytes, d_scratch,
                          scratch_bytes, stream, out);
    if ((int64_t)V * nvec >= (int64_t)1 << 31) return FS_ERR_TOO_LARGE;
    const int n_items = W > 0 ? h_misc[6] : 0;
    const Grain grain = item_grain(NB, W, h_misc[2], t_user, ts_user);
    chunk = grain.T * KB;

    // arena layout, now that the sizes are known.  The value array is followed by 256 zeroed bytes: with no
    // vectors at all every per-vector array has size zero and starts there, so that the kernels' clamped
    // reads of element 0 (column 0, empty mask) stay inside the arena.
    size_t o = fs_align_up((size_t)(W + 1) * 4, 256);
    int32_t *vec_col = (int32_t *)(arena + o); o += fs_align_up((size_t)nvec * 4, 256);
    uint32_t *vec_mask = (uint32_t *)(arena + o); o += fs_align_up((size_t)nvec * 4, 256);
    int32_t *csr_to_slot = (int32_t *)(arena + o); o += fs_align_up((size_t)nnz * 4, 256);
    const size_t vals_bytes = (size_t)V * nvec * 2, vals_padded = fs_align_up(vals_bytes, 256) + 256;
    uint16_t *vals_blk = (uint16_t *)(arena + o); o += vals_padded;
    int4 *blk_desc = (int4 *)(arena + o); o += fs_align_up((size_t)NB * 16, 256);
    int4 *items = (int4 *)(arena + o); o += fs_align_up((size_t)n_items * 16, 256);
    int32_t *item_order = (int32_t *)(arena + o); o += fs_align_up((size_t)n_items * 4, 256);
    int4 *items_by_cost = (int4 *)(arena + o); o += fs_align_up((size_t)n_items * 16, 256);
    int32_t *blk_row_base = (int32_t *)(arena + o); o += fs_align_up((size_t)NB * V * 4, 256);
    uint32_t *blk_row_bits = nullptr;
    if (KB == 32) { blk_row_bits = (uint32_t *)(arena + o); o += fs_align_up((size_t)NB * V * 4, 256); }
    int2 *slot_range = (int2 *)(arena + o); o += fs_align_up((size_t)n_items * 16, 256);  // at most two partial tiles per item
    PlaceOut po{};
    po.vec_col = vec_col; po.vec_mask = vec_mask; po.csr_to_slot = csr_to_slot; po.vals_blk = vals_blk;
    po.blk_desc = blk_desc; po.row_base = blk_row_base; po.row_bits = blk_row_bits;
    po.tail = (uint16_t *)((char *)vals_blk + vals_bytes); po.n_tail = (int)((vals_padded - vals_bytes) / 2); po.n_blocks = NB;
    void *packed = nullptr;
    if (d_vals && nvec > 0 && wants_packed_values(M, nnz, V, KB)) {
        fs_format b{};
        b.n_blocks = NB; b.nvec = nvec; b.nnz = nnz; b.V = V;
        const fs_packed_plan_t pl = fs_packed_plan(&b);
        packed = arena + o;
        po.packed_ofs = (int32_t *)(arena + o + pl.ofs);
        po.packed_m8 = V <= 8 ? (uint8_t *)(arena + o + pl.masks) : nullptr;
        po.packed_m16 = V <= 8 ? nullptr : (uint16_t *)(arena + o + pl.masks);
        po.packed_vals = (uint16_t *)(arena + o + pl.vals);
        o += pl.total;
    }
    int4 *split_windows = (int4 *)(arena + o); o += fs_align_up((size_t)h_misc[5] * 16, 256);

    if (!d_vals || W == 0) FS_HIP(hipMemsetAsync(vals_blk, 0, vals_padded, s));
    if (W > 0) {
        const size_t lds = place_lds_bytes(V, KB);
        const int64_t vb = (int64_t)place_vector_bytes(V);
        const uint16_t *va = (const uint16_t *)d_vals;
        st = launch_units(units_made, [&](int first, unsigned grid) {
#define FS_PLACE(KB32, VT) k_unit_place<KB32, VT><<<grid, 64, lds, s>>>(first, a, up, KB, vb, units, pieces, info, first_vec, win_ptr, blk_ptr, va, po)
            if (KB != 32) FS_PLACE(false, 0);
            else if (V == 4) FS_PLACE(true, 4);
            else if (V == 8) FS_PLACE(true, 8);
            else if (V == 16) FS_PLACE(true, 16);
            else FS_PLACE(true, 0);
#undef FS_PLACE
        });
        if (st != FS_OK) return st;
        if (KB != 32) {
            k_block_row_base<<<grid_for((int64_t)NB * V, 256), 256, 0, s>>>(a, V, blk_desc, NB, vec_col, nvec, blk_row_base);
            FS_LAUNCH_CHECK();
        }
        // With the work list only up to 16 k units, a workgroup a CU: its registers leave half the wavefronts that the shared blocks
        // wait with by themselves (R-MAT of 1 M rows, 100 k units: 72 us together, 45 and 20 apart).
        const bool together = KB == 32 && units_made <= 512 * kSharedPerWave * (kWindowThreads / 64);
        if (nnz > kUnitEntries && !together) {
            const int each = KB == 32 ? kSharedPerWave * kSharedWaves : kSharedPerWave;
            st = launch_units((units_made + each - 1) / each, [&](int first, unsigned grid) {
                if (KB == 32) k_shared_blocks<<<grid, 64 * kSharedWaves, 0, s>>>(first, V, units, units_made, first_vec, win_ptr, blk_ptr, va, po);
                else k_shared_blocks_any<<<grid, 64, 0, s>>>(first, V, KB, units, n_units, first_vec, win_ptr, blk_ptr, va, po);
            }, kSharedWaves);
            if (st != FS_OK) return st;
        }
        // a list too long for one launch to rank may have its hubs in few workgroups; a grid that fills the chip has work enough
        const unsigned shares = n_items > kRankItemsMax ? std::min(std::max(512 / win_grid, 1u), 4u) : 1;
        const ItemFill fill{(int)win_grid, (int)shares, tiles, n_items, grain, item_sums, items, key0, split_windows, slot_range};
        const int shared = nnz > kUnitEntries && together ? grid_for(units_made, kSharedPerWave * (kWindowThreads / 64)) : 0;
        k_finish<<<win_grid * shares + shared, kWindowThreads, 0, s>>>(fill, blk_ptr, W, win_ptr, KB, nvec, K, V, units, units_made, first_vec, va, po);
        FS_LAUNCH_CHECK();
    }

    if (n_items > 0) {
        // launch order: a stable sort by the keys
        if (n_items <= kRankItemsMax) {
            k_item_rank<<<grid_for(n_items, kRankItems), 64 * kRankWaves, 0, s>>>(key0, n_items, items, item_order, items_by_cost);
            FS_LAUNCH_CHECK();
        } else {
            int *hist = scr + sp.hist;
            int32_t *kbuf[2] = {key1, key0};            // pass p reads kbuf[(p + 1) & 1], writes kbuf[p & 1]
            int32_t *vbuf[2] = {item_order, order};     // pass p writes vbuf[p & 1]; the last pass (2) writes item_order
            for (int p = 0; p < 3; p++) {
                if ((st = sort_pass<kKeyDigitBits>((const uint32_t *)kbuf[(p + 1) & 1], p == 0 ? nullptr : vbuf[(p + 1) & 1], n_items, kKeyDigitBits * p,
                                                   kKeyDigitBits, hist, tmp, (uint32_t *)kbuf[p & 1], vbuf[p & 1], s)) != FS_OK)
                    return st;
            }
            k_item_permute<<<grid_for(n_items, 256), 256, 0, s>>>(items, item_order, n_items, items_by_cost);
            FS_LAUNCH_CHECK();
        }
    }
    FS_HIP(hipStreamSynchronize(s));  // (the scratch buffer is the caller's again)

    out->M = M; out->K = K; out->nnz = nnz; out->nvec = nvec; out->W = W;
    out->V = V; out->KB = KB; out->dtype = (int32_t)dtype; out->chunk = chunk;
    out->n_items = n_items; out->n_split_items = h_misc[7]; out->n_split_windows = h_misc[5];
    out->n_cut_items = h_misc[7];
    out->win_ptr = win_ptr; out->vec_col = vec_col; out->vec_mask = vec_mask; out->csr_to_slot = csr_to_slot;
    out->vals_blk = vals_blk; out->blk_desc = (const int32_t *)blk_desc; out->n_blocks = NB;
    out->items = (const int32_t *)items; out->split_windows = (const int32_t *)split_windows;
    out->item_order = item_order; out->items_by_cost = (const int32_t *)items_by_cost;
    out->blk_row_base = blk_row_base;
    out->blk_row_bits = blk_row_bits;
    out->packed = packed;
    out->slot_range = (const int32_t *)slot_range;
    out->arena_used = o;
    return FS_OK;
}

extern "C" fs_status fs_blk_to_csr(const fs_format *fmt, const void *d_blk, void *d_out_csr, void *stream)
{
    if (!fmt || !d_blk || !d_out_csr) return FS_ERR_INVALID_ARG;
    if (fmt->nnz == 0) return FS_OK;
    k_blk_to_csr<uint16_t><<<grid_for(fmt->nnz, 256), 256, 0, (hipStream_t)stream>>>(
        fmt->csr_to_slot, (const uint16_t *)d_blk, (uint16_t *)d_out_csr, fmt->nnz);
    FS_LAUNCH_CHECK();
    return FS_OK;
}

extern "C" fs_status fs_csr_to_blk(const fs_format *fmt, const void *d_vals_csr, void *d_out_blk, void *stream)
{
    if (!fmt || fmt->nvec < 0 || fmt->nnz < 0) return FS_ERR_INVALID_ARG;
    const int64_t n = (int64_t)fmt->V * fmt->nvec;  // elements of the blocked array
    if (n == 0) return FS_OK;
    if (!d_out_blk || ((uintptr_t)d_out_blk & 15) || (fmt->nnz > 0 && !d_vals_csr)) return FS_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    uint16_t *out = (uint16_t *)d_out_blk;
    // By blocks a row slot costs the same whether its row holds an entry or not, entry by entry only entries do.  Entry by entry /
    // by blocks, us, four- / eight- / sixteen-row windows: 4 M rows, 1 M entries 7 / 42, 9.5 / 41, 14 / 40; 4 M rows, 4 M 20 / 45,
    // 29 / 46, 49 / 47; 1 M rows, 1 M 7 / 13.5, 10 / 14, 15.4 / 15.1; 1 M rows, 2 M 12 / 14, 16 / 15, 25 / 16; 1 M rows, 3 M 16 / 15,
    // 22 / 16, 35 / 26: the line is at about eleven entries a block.  Below 640 k row slots launches are the time, and
    // three cost more than one (200 k rows with one entry each 7.3 / 4.8).
    const bool few = fmt->V * fmt->n_blocks > 640 * 1024 && fmt->nnz < 11 * fmt->n_blocks && fmt->csr_to_slot;
    if (!few && fmt->KB == 32 && fmt->blk_desc && fmt->blk_row_bits && fmt->blk_row_base && (fmt->V == 4 || fmt->V == 8 || fmt->V == 16)) {
        const int nb = (int)fmt->n_blocks;
        const unsigned grid = grid_for(nb, 8 * 16 / fmt->V);  // four wavefronts of two rounds
#define FS_TILES(V_) k_csr_to_tiles<V_><<<grid, 256, 0, s>>>((const int4 *)fmt->blk_desc, nb, fmt->blk_row_bits, fmt->blk_row_base, (const uint16_t *)d_vals_csr, (int)fmt->nnz, out)
        if (fmt->V == 4) FS_TILES(4);
        else if (fmt->V == 8) FS_TILES(8);
        else FS_TILES(16);
#undef FS_TILES
        FS_LAUNCH_CHECK();
        return FS_OK;
    }
    // few entries, other block widths and window heights: clear the array, then place entry by entry
    const int64_t n16 = n / 8;  // whole 16-byte pieces; fill kernels, not memset nodes, so the call can be captured
    if (n16 > 0) {
        k_zero16<<<(unsigned)std::min<int64_t>((n16 + 255) / 256, 65536), 256, 0, s>>>((fs_u4 *)out, n16);
        FS_LAUNCH_CHECK();
    }
    if (n16 * 8 < n) {
        k_zero_tail<uint16_t><<<1, 64, 0, s>>>(out, n16 * 8, n);
        FS_LAUNCH_CHECK();
    }
    if (fmt->nnz > 0) {
        k_csr_to_blk<uint16_t><<<grid_for(fmt->nnz, 256), 256, 0, s>>>(fmt->csr_to_slot, (const uint16_t *)d_vals_csr, out,
                                                                         fmt->nnz);
        FS_LAUNCH_CHECK();
    }
    return FS_OK;
}

fs_packed_plan_t fs_packed_plan(const fs_format *f)
{
    fs_packed_plan_t p;
    size_t o = 0;
    p.ofs = o; o += fs_align_up(((size_t)f->n_blocks + 1) * sizeof(int32_t), 256);
    p.tmp = o; o += fs_align_up(scan_tmp_ints(f->n_blocks) * sizeof(int), 256);
    p.masks = o; o += fs_align_up(((size_t)f->nvec + 1) * (f->V <= 8 ? 1 : 2), 256);
    p.vals = o; o += fs_align_up((size_t)f->nnz * 2 + 16, 256);
    p.total = o;
    return p;
}

extern "C" fs_status fs_pack_bytes(const fs_format *fmt, size_t *packed_bytes)
{
    if (!fmt || !packed_bytes || fmt->n_blocks < 0 || fmt->nnz < 0) return FS_ERR_INVALID_ARG;
    *packed_bytes = fs_packed_plan(fmt).total;
    return FS_OK;
}

extern "C" fs_status fs_pack_values(const fs_format *fmt, const void *d_vals_blk, void *d_packed, size_t packed_bytes,
                                    void *stream)
{
    if (!fmt || fmt->n_blocks < 0 || fmt->nnz < 0 || !d_packed || ((uintptr_t)d_packed & 255)) return FS_ERR_INVALID_ARG;
    if (fmt->V < 1 || fmt->V > 16 || fmt->KB != 32) return FS_ERR_UNSUPPORTED;
    const fs_packed_plan_t pl = fs_packed_plan(fmt);
    if (packed_bytes < pl.total) return FS_ERR_BUFFER_TOO_SMALL;
    const uint16_t *vals = (const uint16_t *)(d_vals_blk ? d_vals_blk : fmt->vals_blk);
    if (fmt->nvec > 0 && !vals) return FS_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    unsigned char *buf = (unsigned char *)d_packed;
    int32_t *ofs = (int32_t *)(buf + pl.ofs);
    if (fmt->n_blocks > 0) {
        uint8_t *m8 = fmt->V <= 8 ? (uint8_t *)(buf + pl.masks) : nullptr;
        k_block_nnz<<<grid_for(fmt->n_blocks, 8), 256, 0, s>>>((const int4 *)fmt->blk_desc, fmt->n_blocks, fmt->vec_mask, ofs, m8,
                                                                (uint16_t *)(buf + pl.masks));
        FS_LAUNCH_CHECK();
    }
    fs_status st = scan_exclusive(ofs, fmt->n_blocks, (int *)(buf + pl.tmp), s);
    if (st != FS_OK) return st;
    if (fmt->n_blocks > 0) {
        k_pack<<<grid_for(fmt->n_blocks, 8), 256, 0, s>>>((const int4 *)fmt->blk_desc, fmt->n_blocks, fmt->V, fmt->vec_mask,
                                                             vals, ofs, (uint16_t *)(buf + pl.vals));
        FS_LAUNCH_CHECK();
    }
    return FS_OK;
}

extern "C" int fs_version(void) { return FS_VERSION; }

extern "C" const char *fs_status_string(fs_status s)
{
    switch (s) {
    case FS_OK: return "ok";
    case FS_ERR_INVALID_ARG: return "invalid argument";
    case FS_ERR_INVALID_CSR: return "invalid CSR (column out of range or not strictly ascending in a row)";
    case FS_ERR_UNSUPPORTED: return "unsupported combination of V, KB, dtype or sizes";
    case FS_ERR_BUFFER_TOO_SMALL: return "buffer too small";
    case FS_ERR_TOO_LARGE: return "sizes exceed the 32-bit indices of the format";
    case FS_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}
