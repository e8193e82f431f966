// Edge softmax on gfx950: for every row of A, the softmax of scale * value over the row's stored
// entries, on a value array in the vals_blk layout (the output of fs_sddmm, the input of fs_spmm).
// It is the normalisation step between the two in an attention GNN (the paper's end-to-end
// evaluation, Section 4.4, names the softmax layer without describing a kernel; the definition is
// the usual one).
//
// One wavefront walks one work item (the same items as fs_spmm / fs_sddmm).  Inside an item a window
// appears as a run of consecutive blocks.  A window that lies whole inside the item is finished on
// the spot: row maxima, row sums of exponentials, then the normalised values.  A window cut across
// items leaves (maximum, sum) per row in the workspace slot of each part -- the slots are numbered
// exactly like the partial tiles of fs_spmm -- and a second launch normalises the parts, each of which
// first merges the pairs of all parts of its window in a fixed order.  No atomics: results are
// bit-reproducible.
//
// Lane (block b of a round, row j, group g) handles the eight vectors 8g .. 8g+7 of a row: sixteen bytes of the row-major tile,
// so that a wave-wide load or store moves 1 KB of consecutive blocks (16 / V of them), and one word tells which of the eight A stores.
// kChunk blocks are loaded together: eight with four rows and, for the gradient, with eight, else four.  An item of up to as many is
// read once and stays in registers, its windows side by side; the rows' maxima and sums go from block to block of a window through LDS.  Longer
// items (of R-MAT graphs a fifth of the items with four rows a window, half with eight, 60 % with sixteen) are walked window by window; a window of up to kChunk
// blocks stays in registers between its statistics and its results, a longer one is read twice.  (Steps of whole windows in one loop
// for all items: twice the registers.)
// What bounds it is the chain item -> blocks -> values of the wavefronts and, beside it, the instructions for positions that A does
// not store.  Lognormal graph of 262 k rows, four-row windows (46 k items, 90 MB; 4-byte pieces and a mask per vector): softmax
// 46 -> 37 us, its gradient 69 -> 37;
// stencil of 1 M rows, eight-row windows 71 -> 29 and 92 -> 34.
//
// The same walk serves the gradient of that softmax (BWD): with p the probabilities and g the gradient
// that arrives at them, both in the vals_blk layout,  ds = scale * p * (g - sum over the row of p * g).
// The row statistic is then a plain sum, kept in the second float of a workspace pair.
#include <algorithm>
#include <cmath>

#include "fs_common.h"
#include "fs_tile.h"  // FS_WAVE_SYNC, fs_u4_unaligned

namespace {

template <int DT>
__device__ __forceinline__ float fs_to_float(uint16_t bits)
{
    if (DT == FS_F16) {
        union { uint16_t u; _Float16 h; } c;
        c.u = bits;
        return (float)c.h;
    }
    return __uint_as_float((uint32_t)bits << 16);
}

// (maximum, sum of exp(. - maximum)) of two disjoint sets of scores -> the same for their union
__device__ __forceinline__ void merge_stats(float &top, float &total, float top2, float total2)
{
    const float t = fmaxf(top, top2);
    total = t > -INFINITY ? total * __expf(top - t) + total2 * __expf(top2 - t) : total + total2;  // (zeros, or a NaN)
    top = t;
}

// The value of lane l ^ 1 or l ^ 2: the lanes of a row's four groups are neighbours
template <int X>
__device__ __forceinline__ float quad_xor(float v)
{
    constexpr int ctrl = X == 1 ? 0xB1 : 0x4E;  // quad_perm [1,0,3,2] and [2,3,0,1]
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, false));
}
__device__ __forceinline__ float quad_max(float v)
{
    v = fmaxf(v, quad_xor<1>(v));
    return fmaxf(v, quad_xor<2>(v));
}
__device__ __forceinline__ float quad_sum(float v)
{
    v += quad_xor<1>(v);
    return v + quad_xor<2>(v);
}

// Bit x of m8 as 0 or ~0
__device__ __forceinline__ uint32_t stored(uint32_t m8, int x) { return (uint32_t)__builtin_amdgcn_sbfe((int)m8, x, 1); }

// PARTS = false: statistics of every run, whole windows are normalised, parts of cut windows leave
//                their statistics in the workspace.
// PARTS = true : parts of cut windows are normalised; each merges the statistics its window's parts left in
//                the workspace (a fixed order: deterministic).
// BWD          : the gradient instead: `in` holds the probabilities, `in2` the gradient that arrives at them,
//                the row statistic is sum p * g (second float of a workspace pair), the output
//                scale * p * (g - that sum).
// BITS = false : a format without blk_row_bits; which positions A stores is put together from vec_mask.  (Asked for at run time, the
//                question alone cost sixteen-row windows up to a quarter: their loads no longer travelled together.)
// n_el: elements of the arrays.
template <int DT, int V, bool PARTS, bool BWD, bool BITS>
__global__ void __launch_bounds__(64)
k_edge_softmax(const int4 *__restrict__ items, const int4 *__restrict__ blk_desc,
               const uint32_t *__restrict__ row_bits, const uint32_t *__restrict__ vec_mask, const uint16_t *in, const uint16_t *in2,
               uint16_t *out, int n_el, float *__restrict__ stats, float scale, const int2 *__restrict__ slot_range,
               int n_slots)
{
    constexpr int PER = 16 / V;                      // blocks of a round
    constexpr int ROUNDS = V == 16 || (V == 8 && BWD) ? 4 : 2;  // rounds whose loads are issued together (forward, eight rows, four of them take the
                                                     // registers of half the wavefronts: lognormal graph of 262 k rows 57 us against 66)
    constexpr int kChunk = PER * ROUNDS;             // their blocks
    __shared__ float part[kChunk * V];               // a row's statistic in each block
    __shared__ __attribute__((aligned(16))) uint16_t tile[16 * 32];  // re-lays narrow blocks
    const int lane = threadIdx.x;
    const int4 it = items[blockIdx.x];  // {first block slot, blocks, first workspace slot, first vector}
    const int nblk = it.y;
    if (nblk == 0) return;
    const int g = lane & 3, j = (lane >> 2) % V, b = PER == 1 ? 0 : (lane >> 2) / V;
    // PARTS: where the statistics of the windows of the item's (at most two) parts lie -- slot numbers that
    // follow from the item record alone, so these loads travel together with the descriptors'
    int2 range0 = make_int2(0, 0), range1 = make_int2(0, 0);
    if constexpr (PARTS) {
        range0 = slot_range[min(it.z, n_slots - 1)];
        range1 = slot_range[min(it.z + 1, n_slots - 1)];
    }
    const int4 my_desc = blk_desc[it.x + min(lane, nblk - 1)];  // at most 64 blocks per item
    const uint64_t firsts = __ballot(lane < nblk && (my_desc.y & 512)), lasts = __ballot(lane < nblk && (my_desc.y & 256));

    // Eight positions of a row: what A stores of them, the values and (BWD) the gradient.
    struct Eight {
        int s, kb;     // first vector and width of the block, 0: none
        uint32_t m8;
        fs_frag v, d;
    };
    // block i of the item (none from `end` on); the bits do not depend on the descriptor, so they are under way beside it
    auto bits_of = [&](int i, int end) -> uint32_t { return BITS && i < end ? row_bits[(int64_t)(it.x + i) * V + j] >> (8 * g) & 0xFFu : 0u; };
    auto values_of = [&](const uint16_t *from, const Eight &x) -> fs_frag {
        // Narrow blocks: what follows the row, or the block, is read along with it and not looked at; at the end of the array it is not there.
        const uint32_t at = (uint32_t)V * x.s + j * x.kb + 8 * g;  // (up to 2^31 elements)
        fs_frag r;
        r.u = fs_u4{0u, 0u, 0u, 0u};
        if (at + 8 <= (uint32_t)n_el) {
            r.u = *reinterpret_cast<const fs_u4_unaligned *>(from + at);
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++) r.e[k] = at + k < (uint32_t)n_el ? from[at + k] : (uint16_t)0;
        }
        return r;
    };
    auto fetch = [&](Eight &x, int i, int end) {
        const int ic = min(i, nblk - 1);
        if constexpr (PER == 1) {  // the same block for all lanes
            x.s = __builtin_amdgcn_readlane(my_desc.x, ic);
            x.kb = __builtin_amdgcn_readlane(my_desc.y, ic) & 255;
        } else {
            x.s = __shfl(my_desc.x, ic, 64);
            x.kb = __shfl(my_desc.y, ic, 64) & 255;
        }
        if (i >= end) x.kb = 0;
        if constexpr (!BITS) {
#pragma unroll
            for (int k = 0; k < 8; k++) x.m8 |= 8 * g + k < x.kb ? (vec_mask[x.s + 8 * g + k] >> j & 1u) << k : 0u;
        }
        x.v = values_of(in, x);
        if constexpr (BWD) x.d = values_of(in2, x);
    };
    auto score = [&](const Eight &x, int k) -> float {  // scaled, -infinity where A stores nothing
        const uint32_t keep = stored(x.m8, k);
        return __uint_as_float((keep & __float_as_uint(scale * fs_to_float<DT>(x.v.e[k]))) | (~keep & 0xFF800000u));
    };
    auto dot = [&](const Eight &x) -> float {  // sum of p * g
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint32_t keep = stored(x.m8, k);
            t = fmaf(__uint_as_float(keep & __float_as_uint(fs_to_float<DT>(x.v.e[k]))), __uint_as_float(keep & __float_as_uint(fs_to_float<DT>(x.d.e[k]))), t);
        }
        return t;
    };
    // Results of a round to their blocks; positions that A does not store get +0.0.
    auto store = [&](const Eight &x, const float (&y)[8], bool mine) {
        fs_frag o;
        o.u = fs_u4{fs_pack2<DT>(y[0], y[1]), fs_pack2<DT>(y[2], y[3]), fs_pack2<DT>(y[4], y[5]), fs_pack2<DT>(y[6], y[7])};
        const int kb = mine ? x.kb : 0;
        uint16_t *blk = out + (int64_t)V * x.s;
        if (kb == 32) *reinterpret_cast<fs_u4_unaligned *>(blk + j * 32 + 8 * g) = o.u;  // (four rows: blocks begin on eight bytes; the array on any element)
        const bool narrow = kb > 0 && kb < 32;
        if (!__ballot(narrow)) return;
        uint16_t *mine_at = tile + b * (32 * V);
        if (narrow) {
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (8 * g + k < kb) mine_at[j * kb + 8 * g + k] = o.e[k];
        }
        FS_WAVE_SYNC();
        const int at = 8 * (j * 4 + g);
        if (narrow) {
            if (at + 8 <= V * kb) *reinterpret_cast<fs_u4_unaligned *>(blk + at) = *reinterpret_cast<const fs_u4 *>(mine_at + at);
            else if (V == 4 && at < V * kb) *reinterpret_cast<fs_u2_unaligned *>(blk + at) = *reinterpret_cast<const fs_u2 *>(mine_at + at);  // odd widths
        }
        FS_WAVE_SYNC();
    };
    // exp(v - top) / total, one score at a time.  The fast exponential returns zero where the result would be a subnormal fp32 number, a
    // range bf16 still represents: far below the maximum, evaluate e^(x+40) and scale by e^-40 (the
    // multiplication keeps subnormal results).
    auto probability = [&](float v, float top, float inv) -> float {
        const float x = v - top;
        const float p = x < -80.f ? __expf(x + 40.f) * 4.24835425529158899533e-18f : __expf(x);
        return v > -INFINITY ? p * inv : 0.f;
    };
    auto emit = [&](const Eight &x, float top, float total, bool mine) {
        float y[8];
        if constexpr (BWD) {
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const uint32_t keep = stored(x.m8, k);
                y[k] = __uint_as_float(keep & __float_as_uint(scale * fs_to_float<DT>(x.v.e[k]) * (fs_to_float<DT>(x.d.e[k]) - total)));
            }
        } else {
            const float inv = total > 0.f ? 1.f / total : 0.f;
#pragma unroll
            for (int k = 0; k < 8; k++) y[k] = probability(score(x, k), top, inv);
        }
        store(x, y, mine);
    };
    auto pair_to_workspace = [&](int slot, float top, float total) {
        float *st = stats + (int64_t)slot * 2 * V;
        st[j] = BWD ? 0.f : top;
        st[V + j] = total;
    };
    // over the lanes that share row j
    auto reduce_row = [&](float &top, float &total) {
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            if (o >= 4 && o < 4 * V) continue;
            if constexpr (BWD) total += __shfl_xor(total, o, 64);
            else merge_stats(top, total, __shfl_xor(top, o, 64), __shfl_xor(total, o, 64));
        }
    };

    if constexpr (PARTS) {
        // the item's first run if its window begins before the item, and its last if its window goes on behind it; the
        // parts of a window left their pairs in consecutive workspace slots.  Lane (b, j, g) merges the pairs of row j over
        // the parts 4b + g, 4b + g + 64/V, ... and the lanes of a row are merged by shuffles: a fixed order, deterministic.
        const bool head = !(firsts & 1), tail = !(lasts >> (nblk - 1) & 1);
        const int head_end = lasts ? (int)__builtin_ctzll(lasts) + 1 : nblk;           // blocks of the first run
        const int tail_at = firsts ? 63 - (int)__builtin_clzll(firsts) : 0;            // where the last run begins
        for (int run = 0; run < 2; run++) {
            if (run == 0 ? !head : !tail || (head && head_end == nblk)) continue;  // (a part inside its window is the first run)
            const int2 rg = run == 0 || !head ? range0 : range1;
            const float *st = stats + (int64_t)rg.x * 2 * V;
            float top = -INFINITY, total = 0.f;
            for (int k = 4 * b + g; k < rg.y; k += 64 / V) {
                if constexpr (BWD) total += st[k * 2 * V + V + j];
                else merge_stats(top, total, st[k * 2 * V + j], st[k * 2 * V + V + j]);
            }
            reduce_row(top, total);
            const int end = run == 0 ? head_end : nblk;
            for (int c = run == 0 ? 0 : tail_at; c < end; c += kChunk) {
                Eight x[ROUNDS];
#pragma unroll
                for (int r = 0; r < ROUNDS; r++) {
                    if (c + r * PER >= end) break;
                    const int i = c + r * PER + b;
                    x[r].m8 = bits_of(i, end);
                    fetch(x[r], i, end);
                }
#pragma unroll
                for (int r = 0; r < ROUNDS; r++) {
                    if (c + r * PER >= end) break;
                    emit(x[r], top, total, true);
                }
            }
        }
        return;
    }
    if (nblk <= kChunk) {
        Eight x[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) x[r].m8 = bits_of(r * PER + b, nblk);
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            if (r * PER >= nblk) break;
            fetch(x[r], r * PER + b, nblk);
        }
        // the lane's window in a round: its blocks of the item, and whether they are all of it
        auto run_of = [&](int i, int &lo, int &hi) -> bool {
            const uint64_t before = firsts & ((2ull << i) - 1), after = lasts >> i;
            lo = before ? 63 - (int)__builtin_clzll(before) : 0;
            hi = after ? i + (int)__builtin_ctzll(after) : nblk - 1;
            return before && after;
        };
        auto over_run = [&](int i, float own, auto combine) -> float {  // of what every block's lanes left in part[]
            int lo, hi;
            run_of(i, lo, hi);
            if (lo == hi) return own;
            float t = part[lo * V + j];
            for (int k = lo + 1; k <= hi; k++) t = combine(t, part[k * V + j]);
            return t;
        };
        float top[ROUNDS], total[ROUNDS], e[ROUNDS][8];
        // No score is so far below its row's maximum, and none so large or no number, that the exponential needs care: known from
        // the largest magnitude among the values (they compare like whole numbers) without a look at each difference.
        bool plain = true;
        if constexpr (!BWD) {
#pragma unroll
            for (int r = 0; r < ROUNDS; r++) {
                if (r * PER >= nblk) break;
                float t = -INFINITY;
                uint32_t largest = 0;
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    e[r][k] = score(x[r], k);
                    t = fmaxf(t, e[r][k]);
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t magnitude = x[r].v.u[k] & 0x7FFF7FFFu;
                    typedef uint16_t two __attribute__((ext_vector_type(2)));
                    const two m = __builtin_elementwise_max(__builtin_bit_cast(two, magnitude), __builtin_bit_cast(two, largest));
                    largest = __builtin_bit_cast(uint32_t, m);
                }
                plain = plain && fabsf(scale) * fs_to_float<DT>((uint16_t)max(largest & 0xFFFF, largest >> 16)) <= 39.f;
                top[r] = quad_max(t);
                if (g == 0) part[(r * PER + b) * V + j] = top[r];
            }
            FS_WAVE_SYNC();
#pragma unroll
            for (int r = 0; r < ROUNDS; r++) {
                if (r * PER >= nblk) break;
                const int i = min(r * PER + b, nblk - 1);
                top[r] = over_run(i, top[r], [](float a, float c) { return fmaxf(a, c); });
            }
            FS_WAVE_SYNC();
        }
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            if (r * PER >= nblk) break;
            if constexpr (BWD) {
                total[r] = dot(x[r]);
            } else {
                const float from = top[r] > -INFINITY ? top[r] : 0.f;  // (nothing stored, or minus infinity only: all exponentials are zero)
                float sum = 0.f;
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    e[r][k] = __expf(e[r][k] - from);  // exp(-inf) = 0 where nothing is stored
                    sum += e[r][k];
                }
                total[r] = sum;
            }
            total[r] = quad_sum(total[r]);
            if (g == 0) part[(r * PER + b) * V + j] = total[r];
        }
        FS_WAVE_SYNC();
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            if (r * PER >= nblk) break;
            const int i = min(r * PER + b, nblk - 1);
            total[r] = over_run(i, total[r], [](float a, float c) { return a + c; });
        }
        const bool fast = !BWD && !__ballot(!plain);
#pragma unroll
        for (int r = 0; r < ROUNDS; r++) {
            if (r * PER >= nblk) break;
            const int i = r * PER + b;
            int lo, hi;
            const bool whole = run_of(min(i, nblk - 1), lo, hi);
            if (fast) {
                const float inv = total[r] > 0.f ? 1.f / total[r] : 0.f;
#pragma unroll
                for (int k = 0; k < 8; k++) e[r][k] *= inv;
                store(x[r], e[r], whole);
            } else {
                emit(x[r], BWD ? 0.f : top[r], total[r], whole);
            }
            // a part's rows, by the lanes of its first block; it is the second part of the item if the first begins before it
            if (!whole && i == lo && g == 0) pair_to_workspace(it.z + (lo > 0 && !(firsts & 1) ? 1 : 0), BWD ? 0.f : top[r], total[r]);
        }
        return;
    }
    int slot = it.z;
    for (int a = 0; a < nblk;) {  // run by run
        const uint64_t after = lasts >> a;
        const int end = after ? a + (int)__builtin_ctzll(after) + 1 : nblk;
        const bool whole = after && (firsts >> a & 1);
        float top = -INFINITY, total = 0.f;
        Eight x[ROUNDS];
        for (int c = a; c < end; c += kChunk) {
#pragma unroll
            for (int r = 0; r < ROUNDS; r++) {
                if (c + r * PER >= end) break;
                const int i = c + r * PER + b;
                x[r].m8 = bits_of(i, end);
                fetch(x[r], i, end);
            }
#pragma unroll
            for (int r = 0; r < ROUNDS; r++) {
                if (c + r * PER >= end) break;
                if constexpr (BWD) {
                    total += dot(x[r]);
                } else {
                    float v[8], t = -INFINITY;
                    const float was = top;
#pragma unroll
                    for (int k = 0; k < 8; k++) {
                        v[k] = score(x[r], k);
                        t = fmaxf(t, v[k]);
                    }
                    // (a NaN, which no maximum shows, has to reach the sum even where it is all that the lane holds)
                    top = fmaxf(t, top);
                    const float from = top > -INFINITY ? top : 0.f;
                    total *= __expf(was - from);
#pragma unroll
                    for (int k = 0; k < 8; k++) total += __expf(v[k] - from);  // exp(-inf) = 0 where nothing is stored
                }
            }
        }
        reduce_row(top, total);
        if (!whole) {
            if (g == 0 && b == 0) pair_to_workspace(slot, top, total);
            slot++;
        } else {
            for (int c = a; c < end; c += kChunk) {
#pragma unroll
                for (int r = 0; r < ROUNDS; r++) {
                    if (c + r * PER >= end || end - a <= kChunk) break;
                    const int i = c + r * PER + b;
                    x[r].m8 = bits_of(i, end);
                    fetch(x[r], i, end);
                }
#pragma unroll
                for (int r = 0; r < ROUNDS; r++) {
                    if (c + r * PER >= end) break;
                    emit(x[r], top, total, true);
                }
            }
        }
        a = end;
    }
}

template <int DT, int V, bool BWD, bool BITS>
fs_status launch_with(const fs_format *f, const uint16_t *in, const uint16_t *in2, uint16_t *out, float scale, float *stats,
                 hipStream_t st)
{
    if (f->n_items == 0) return FS_OK;
    // The work list in launch order: the items that hold a part of a cut window come first (n_cut_items of
    // them), the whole windows after them, costliest first.  The second launch only needs the former.
    const int4 *items = (const int4 *)f->items_by_cost;
    const int n_items = (int)f->n_items;
    const int n_el = (int)(V * f->nvec);
    k_edge_softmax<DT, V, false, BWD, BITS><<<(unsigned)n_items, 64, 0, st>>>(items, (const int4 *)f->blk_desc, f->blk_row_bits, f->vec_mask, in, in2, out, n_el, stats, scale,
                                                                        (const int2 *)f->slot_range, (int)f->n_split_items);
    FS_LAUNCH_CHECK();
    const int n_cut = (int)std::min<int64_t>(f->n_cut_items, f->n_items);
    if (f->n_split_windows > 0 && n_cut > 0) {
        k_edge_softmax<DT, V, true, BWD, BITS><<<(unsigned)n_cut, 64, 0, st>>>(items, (const int4 *)f->blk_desc, f->blk_row_bits, f->vec_mask, in, in2, out, n_el, stats, scale,
                                                                         (const int2 *)f->slot_range, (int)f->n_split_items);
        FS_LAUNCH_CHECK();
    }
    return FS_OK;
}

template <int DT, int V, bool BWD>
fs_status launch(const fs_format *f, const uint16_t *in, const uint16_t *in2, uint16_t *out, float scale, float *stats,
                 hipStream_t st)
{
    return f->blk_row_bits ? launch_with<DT, V, BWD, true>(f, in, in2, out, scale, stats, st)
                           : launch_with<DT, V, BWD, false>(f, in, in2, out, scale, stats, st);
}

template <bool BWD>
fs_status launch_any(const fs_format *f, const uint16_t *in, const uint16_t *in2, uint16_t *out, float scale, float *stats,
                     hipStream_t st)
{
    if (f->dtype == FS_F16) {
        if (f->V == 4) return launch<FS_F16, 4, BWD>(f, in, in2, out, scale, stats, st);
        if (f->V == 8) return launch<FS_F16, 8, BWD>(f, in, in2, out, scale, stats, st);
        if (f->V == 16) return launch<FS_F16, 16, BWD>(f, in, in2, out, scale, stats, st);
    } else if (f->dtype == FS_BF16) {
        if (f->V == 4) return launch<FS_BF16, 4, BWD>(f, in, in2, out, scale, stats, st);
        if (f->V == 8) return launch<FS_BF16, 8, BWD>(f, in, in2, out, scale, stats, st);
        if (f->V == 16) return launch<FS_BF16, 16, BWD>(f, in, in2, out, scale, stats, st);
    }
    return FS_ERR_UNSUPPORTED;
}

}  // namespace

fs_status fs_edge_softmax_launch(const fs_format *f, const void *d_in, void *d_out, float scale, void *d_work,
                                 hipStream_t st)
{
    return launch_any<false>(f, (const uint16_t *)d_in, nullptr, (uint16_t *)d_out, scale, (float *)d_work, st);
}

fs_status fs_edge_softmax_backward_launch(const fs_format *f, const void *d_p, const void *d_g, void *d_out, float scale,
                                          void *d_work, hipStream_t st)
{
    return launch_any<true>(f, (const uint16_t *)d_p, (const uint16_t *)d_g, (uint16_t *)d_out, scale, (float *)d_work, st);
}
