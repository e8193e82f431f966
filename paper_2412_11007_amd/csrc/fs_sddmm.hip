// SDDMM on the CDNA4 matrix cores over the row-window format (paper Section 3.4).
//
// For every block of up to 32 nonzero vectors of a window the kernel computes
// the V x 32 tile  X[window rows, :] * Y[vector columns, :]^T  and writes it,
// masked by the sparsity pattern, straight into the value layout fs_spmm reads
// (the role the paper gives its Algorithm 1).
//
// As in SpMM the operands are swapped (Section 3.2): gathered Y rows are the left operand (16 vectors x 32
// features), the window's X rows the right operand (32 features x 16 rows, rows >= V zero).
// Vector c of a block is placed on row 8*(i/4)+4t+(i%4) -> i of tile t, so that
// after both tiles a lane holds the eight consecutive vectors 8g..8g+7 of one
// window row: exactly 16 contiguous bytes of the row-major value tile.
//
// The contraction runs over the feature dimension d, which is contiguous in the rows of both X and Y (the
// alignment the paper points out at the end of Section 3.4), so the matrix-core operand can be loaded
// straight from memory, 16 bytes per lane.  In operand layout neighbouring lanes read different rows, and the
// vector-memory unit then takes a cycle per lane: 64-70 cycles per wave-wide load, 9 TB/s over the chip, however
// often the rows hit a cache.  With neighbouring lanes on one row a load takes 18-24 cycles.  So for d > 32
// the rows are gathered row by row like those of SpMM and turned into operand layout in LDS (R-MAT of 65 k rows,
// d = 128: 38 -> 20 us; lognormal graph of 262 k rows, d = 256: 560 -> 389 us, 7.0 TB/s of rows that miss the
// L2s).  For d <= 32 a row is half a cache line at most, the loads are few and the L2s set the time; the detour
// costs 2-5 % there and is left out.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "fs_common.h"
#include "fs_tile.h"

namespace {

// The scores of one block, masked by the pattern, to memory.  Lane (j, g): acc[t][e] is the score of window row
// j and vector 8g + 4t + e; bit c of bits says whether row j stores vector c, rbase is the CSR position of row j's first
// entry in the block, blk the block's place in the value array (null: CSR order only).
template <int DT, int V, bool CSR>
__device__ __forceinline__ void fs_store_scores(const fs_f4 (&acc)[2], uint32_t bits, int kb, int rbase, int lane, uint16_t *tile,
                                                uint16_t *__restrict__ blk, uint16_t *__restrict__ out_csr)
{
    const int j = lane & 15, g = lane >> 4;
    fs_frag o;
    o.u.x = fs_pack2<DT>(acc[0][0], acc[0][1]);
    o.u.y = fs_pack2<DT>(acc[0][2], acc[0][3]);
    o.u.z = fs_pack2<DT>(acc[1][0], acc[1][1]);
    o.u.w = fs_pack2<DT>(acc[1][2], acc[1][3]);
    const uint32_t mine = bits >> (8 * g);  // bit x: vector 8g + x
    uint32_t keep[4];  // 0xFFFF per stored position, else 0: sign-extended single bits
#pragma unroll
    for (int p = 0; p < 4; p++)
        keep[p] = ((uint32_t)__builtin_amdgcn_sbfe((int)mine, 2 * p, 1) & 0xFFFFu) |
                  ((uint32_t)__builtin_amdgcn_sbfe((int)mine, 2 * p + 1, 1) & 0xFFFF0000u);
    o.u.x &= keep[0]; o.u.y &= keep[1]; o.u.z &= keep[2]; o.u.w &= keep[3];
    if constexpr (CSR) {
        if (j < V) {
            // CSR order: the entries of row j inside this block are consecutive positions, in vector order
            int pos = rbase + __popc(bits & ((1u << (8 * g)) - 1u));
#pragma unroll
            for (int x = 0; x < 8; x++) {
                if ((mine >> x) & 1u) out_csr[pos++] = o.e[x];
            }
        }
        if (!blk) return;
    }
    if (kb == 32) {
        if (j < V) *reinterpret_cast<fs_u4 *>(blk + j * 32 + 8 * g) = o.u;
    } else {
        // narrow last block of the window (row stride kb): gather the V x kb tile in LDS,
        // then store its V*kb contiguous values 16 bytes per lane
        if (j < V) {
#pragma unroll
            for (int x = 0; x < 8; x++) {
                const int c = 8 * g + x;
                if (c < kb) tile[j * kb + c] = o.e[x];
            }
        }
        FS_WAVE_SYNC();
        if (lane * 8 + 8 <= V * kb)
            *reinterpret_cast<fs_u4 *>(blk + 8 * lane) = *reinterpret_cast<const fs_u4 *>(tile + 8 * lane);
        else if (V == 4 && lane * 8 < V * kb)  // V = 4, odd width: the last piece holds four values
            *reinterpret_cast<uint2 *>(blk + 8 * lane) = *reinterpret_cast<const uint2 *>(tile + 8 * lane);
        FS_WAVE_SYNC();
    }
}

// Bytes between rows; BIG takes any pitch, up to rows of 4 GiB and more.
template <bool BIG>
using fs_pitch = std::conditional_t<BIG, uint64_t, uint32_t>;

// Which block slots a wavefront takes; false: none.  With `items`, those of a work item, in the launch order of
// SpMM: parts of hub windows by column, placed per XCD, so that they share rows of Y in L2 (R-MAT of 262 k rows,
// d = 128: 108 -> 75 us).  Without, G consecutive slots straight from the block table, whatever windows they
// belong to -- a block of scores depends on nothing but its own descriptor, and the item record would be one
// more dependent load.  One wavefront per workgroup: wavefronts share nothing, and a workgroup keeps its slots
// until its slowest wavefront is done.
__device__ __forceinline__ bool fs_sddmm_unit(const int4 *__restrict__ items, int n_items, int slice, int n_swz, int n_blocks, int G,
                                              int &first, int &nblk)
{
    if (items) {
        const int turn = fs_launch_turn<1>(blockIdx.x, slice, n_swz);
        if (turn >= n_items) return false;
        const int4 it = items[turn];
        first = it.x;
        nblk = it.y;
        return nblk > 0;
    }
    first = blockIdx.x * G;
    nblk = min(G, n_blocks - first);
    return nblk > 0;
}

// d > 32.  KS = 32-feature steps of the contraction per chunk of 32 * KS features (one chunk for d <= 32 * KS, else d is
// walked in several); BB = blocks per step, BB * KS = 4: a step gathers its rows in eight wave-wide loads.  KS = 8 (BB = 1)
// gathers whole rows of up to 512 bytes in sixteen: the two halves of a row are not fetched at different times, and blocks of
// one window keep their rows of X, which chunks read anew (lognormal graph of 262 k rows, four-row windows, d = 256: 424 -> 389 us; see
// the launch for where it is used).
// CSR: also (or only) write the scores in CSR order; kept out of the plain instantiation, whose registers it
// would cost.  BIG: X or Y spans 4 GiB or more.
template <int DT, int V, int KS, int BB, bool CHUNKS, bool BIG, bool CSR>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(KS > 4 ? 2 : 4)))
k_sddmm(const int4 *__restrict__ items, int n_items, int slice, int n_swz, int n_blocks, int G, const int4 *__restrict__ blk_desc,
        const int32_t *__restrict__ vec_col, const uint32_t *__restrict__ row_bits, int nvec,
        const uint16_t *__restrict__ X, int64_t ldx, const uint16_t *__restrict__ Y, int64_t ldy, int d,
        uint16_t *__restrict__ out, int64_t M, uint16_t *__restrict__ out_csr, const int32_t *__restrict__ row_base)
{
    constexpr int LPR = 4 * KS;       // lanes that share one gathered row (16 bytes each)
    constexpr int RPI = 64 / LPR;     // rows per wave-wide load
    constexpr int LPB = 32 / RPI;     // wave-wide loads per block
    constexpr int NLD = BB * LPB;     // ... and per step
    constexpr int NF = 32 * KS;       // features per chunk
    constexpr int RS = NF * 2 + 16;   // LDS row stride: an odd number of 16-byte pieces, so that the sixteen rows of
                                      // an operand read start in sixteen different groups of four banks
    __shared__ __attribute__((aligned(16))) unsigned char lds[BB * 32 * RS];
    __shared__ __attribute__((aligned(16))) uint16_t tile[V * 32];  // re-lays the scores of a narrow block before they are stored

    const int lane = threadIdx.x;
    int first, nblk;  // first block slot of this wavefront, and how many
    if (!fs_sddmm_unit(items, n_items, slice, n_swz, n_blocks, G, first, nblk)) return;
    const int j = lane & 15, g = lane >> 4;
    const unsigned char *Xb = reinterpret_cast<const unsigned char *>(X);
    const unsigned char *Yb = reinterpret_cast<const unsigned char *>(Y);
    const fs_pitch<BIG> ldx2 = (fs_pitch<BIG>)ldx * 2, ldy2 = (fs_pitch<BIG>)ldy * 2;  // bytes between rows

    // descriptors of the unit's blocks (at most 64), one per lane
    const int4 my_desc = blk_desc[first + min(lane, nblk - 1)];

    // Gather geometry.  LDS row p of a block's tile holds vector 8*((p%16)/4) + 4*(p/16) + p%4: the sixteen rows
    // of an operand tile are then neighbours.  Lane l of load k serves LDS row k*RPI + l/LPR.
    const int g_row = lane / LPR, g_piece = lane % LPR;
    auto vector_of = [](int p) -> int { return 8 * ((p & 15) >> 2) + 4 * (p >> 4) + (p & 3); };
    unsigned char *lds_wr = lds + g_row * RS + g_piece * 16;        // + k*RPI*RS per load
    const unsigned char *lds_rd = lds + j * RS + g * 16;            // + (b*32 + 16*t)*RS + 64*ks per read
    // features past d: the lane does not read past the row (it repeats the row's last piece), and LDS holds zeros there
    const int n_chunks = CHUNKS ? (d + NF - 1) / NF : 1;
    if (!CHUNKS && d < NF) {  // zero what no lane will write
        for (int o = lane * 16; o < BB * 32 * RS; o += 64 * 16) *reinterpret_cast<fs_u4 *>(lds + o) = fs_u4{0u, 0u, 0u, 0u};
        FS_WAVE_SYNC();
    }

    // With sixteen lanes per row every group of 16 lanes wants one index per load: lane i of a group holds the
    // index for load i and a DPP move hands it out.  Shorter rows keep the indices one per vector.
    // Both loads take a scalar base and a small lane offset.  Lanes past the block's width repeat its last vector;
    // the slot of an empty window reads some valid element.
    const uint32_t v_byte = 4 * (LPR == 16 ? vector_of(((lane & 15) * RPI + g_row) & 31) : (lane & 31));
    auto load_cols = [&](const BlockDesc &b) -> int {
        const char *base = reinterpret_cast<const char *>(vec_col + min(b.s, nvec - 1));
        return *reinterpret_cast<const int32_t *>(base + min(v_byte, 4u * (uint32_t)(max(b.kb, 1) - 1)));
    };
    // occupancy of the lane's window row in block i of the unit (any row's for lanes past V, which store nothing)
    auto load_bits = [&](int i) -> uint32_t { return row_bits[(int64_t)(first + min(i, nblk - 1)) * V + (j & (V - 1))]; };
    auto load_base = [&](int i) -> int { return CSR ? row_base[(int64_t)(first + min(i, nblk - 1)) * V + (j & (V - 1))] : 0; };
    fs_u4 stage[NLD];
    uint32_t grow[NLD];  // byte offsets of the rows this lane gathers in a step (row numbers if BIG)
    auto rows_of = [&](const int (&cols)[BB]) {
        fs_for_each_index([&](auto k_) {
            constexpr int k = decltype(k_)::value, b = k / LPB, l = k % LPB;
            int idx;
            if constexpr (LPR == 16) idx = fs_row_bcast<l>(cols[b]);
            else idx = __shfl(cols[b], vector_of(l * RPI + g_row), 64);
            grow[k] = BIG ? (uint32_t)idx : fs_mul24((uint32_t)idx, ldy2);
        }, std::make_integer_sequence<int, NLD>{});
    };
    auto gather = [&](int f_base) {
        const int f = max(min(f_base + g_piece * 8, d - 8), 0);
#pragma unroll
        for (int k = 0; k < NLD; k++)
            stage[k] = *reinterpret_cast<const fs_u4 *>(Yb + (BIG ? (uint64_t)grow[k] * ldy2 : (uint64_t)grow[k]) + 2 * (uint32_t)f);
    };
    // X operand of a block: lane (j, g) holds X[w*V + j][f_base + 32*ks + 8g .. +7]; rows past V or M are zero
    auto load_x = [&](int w, int f_base, fs_frag (&x)[KS]) {
        const int64_t row = (int64_t)w * V + j;
        const bool ok = j < V && row < M;
        const uint64_t off = BIG ? (uint64_t)row * ldx2 : (uint64_t)fs_mul24((uint32_t)row, ldx2);
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
            const int f = f_base + 32 * ks + 8 * g;
            x[ks].u = fs_u4{0u, 0u, 0u, 0u};
            if (ok && f < d) x[ks].u = *reinterpret_cast<const fs_u4 *>(Xb + off + 2 * (uint32_t)f);
        }
    };

    const int n_steps = (nblk + BB - 1) / BB;
    BlockDesc cur[BB], nxt[BB];
    int col[BB];
    uint32_t bits[BB], bits_n[BB];
    int rbase[BB], rbase_n[BB];  // CSR position of window row j's first entry in the block (CSR-order output only)
    fs_frag xf[BB][KS];
    auto load_xs = [&](const BlockDesc (&blk)[BB], int f_base) {
#pragma unroll
        for (int b = 0; b < BB; b++) load_x(blk[b].w, f_base, xf[b]);
    };
    // the indices, row occupancies and CSR positions of a later step, loaded ahead (read where they are used, the
    // positions cost a memory round trip per step: uniform matrix of 1 M rows with three entries each, d = 64, CSR
    // order: 104 -> 83 us)
    auto look_ahead = [&](int st) {
#pragma unroll
        for (int b = 0; b < BB; b++) {
            nxt[b] = fs_item_block(my_desc, st * BB + b, nblk);
            col[b] = load_cols(nxt[b]);
            bits_n[b] = load_bits(st * BB + b);
            rbase_n[b] = load_base(st * BB + b);
        }
    };
#pragma unroll
    for (int b = 0; b < BB; b++) {
        cur[b] = fs_item_block(my_desc, b, nblk);
        col[b] = load_cols(cur[b]);
        bits[b] = load_bits(b);
        rbase[b] = load_base(b);
    }
    rows_of(col);
    gather(0);
    if constexpr (!CHUNKS) load_xs(cur, 0);
    look_ahead(1);
    for (int st = 0; st < n_steps; st++) {
        const bool more = st + 1 < n_steps;
        fs_f4 acc[BB][2];
#pragma unroll
        for (int b = 0; b < BB; b++)
#pragma unroll
            for (int t = 0; t < 2; t++) acc[b][t] = fs_f4{0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < n_chunks; c++) {
            if constexpr (CHUNKS) load_xs(cur, c * NF);
            // the gathered rows go to LDS (this is where the wave waits for the gather), and the next gather starts
            if (c * NF + g_piece * 8 < d) {
#pragma unroll
                for (int k = 0; k < NLD; k++) *reinterpret_cast<fs_u4 *>(lds_wr + k * RPI * RS) = stage[k];
            } else if (CHUNKS) {
#pragma unroll
                for (int k = 0; k < NLD; k++) *reinterpret_cast<fs_u4 *>(lds_wr + k * RPI * RS) = fs_u4{0u, 0u, 0u, 0u};
            }
            if (CHUNKS && c + 1 < n_chunks) gather((c + 1) * NF);
            else if (more) {
                rows_of(col);
                gather(0);
            }
            FS_WAVE_SYNC();
#pragma unroll
            for (int b = 0; b < BB; b++)
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int ks = 0; ks < KS; ks++) {
                        fs_frag y;
                        y.u = *reinterpret_cast<const fs_u4 *>(lds_rd + (b * 32 + 16 * t) * RS + 64 * ks);
                        acc[b][t] = fs_mfma_16x16x32<DT>(y, xf[b][ks], acc[b][t]);
                    }
            FS_WAVE_SYNC();
        }
#pragma unroll
        for (int u = 0; u < BB; u++) {
            const int kb = cur[u].kb;
            if (kb <= 0) continue;
            fs_store_scores<DT, V, CSR>(acc[u], bits[u], kb, rbase[u], lane, tile, out ? out + (int64_t)V * cur[u].s : nullptr, out_csr);
        }
        if (more) {
#pragma unroll
            for (int b = 0; b < BB; b++) {
                // blocks of one window keep its rows of X (in operand layout, so a load of half a step's gather)
                if (!CHUNKS && nxt[b].w != cur[b].w) load_x(nxt[b].w, 0, xf[b]);
                cur[b] = nxt[b];
                bits[b] = bits_n[b];
                rbase[b] = rbase_n[b];
            }
            look_ahead(st + 2);
        }
    }
}

// d <= 32: a round of four blocks loads every block's indices, masks and rows of X, then every row of Y, straight
// in operand layout (see above), so that it costs two memory round trips however many blocks it holds.
template <int DT, int V, bool BIG, bool CSR>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(CSR ? 5 : 6)))
k_sddmm_short(const int4 *__restrict__ items, int n_items, int slice, int n_swz, int n_blocks, int G, const int4 *__restrict__ blk_desc,
        const int32_t *__restrict__ vec_col, const uint32_t *__restrict__ row_bits, int /* as k_sddmm, which the launch shares its arguments with */,
        const uint16_t *__restrict__ X, int64_t ldx, const uint16_t *__restrict__ Y, int64_t ldy, int d,
        uint16_t *__restrict__ out, int64_t M, uint16_t *__restrict__ out_csr, const int32_t *__restrict__ row_base)
{
    constexpr int BB = 4;  // blocks per round
    __shared__ __attribute__((aligned(16))) uint16_t lds[V * 32];  // re-lays the scores of a narrow block before they are stored

    const int lane = threadIdx.x;
    int first, nblk;
    if (!fs_sddmm_unit(items, n_items, slice, n_swz, n_blocks, G, first, nblk)) return;
    const int j = lane & 15, g = lane >> 4;
    const unsigned char *Xb = reinterpret_cast<const unsigned char *>(X);
    const unsigned char *Yb = reinterpret_cast<const unsigned char *>(Y);
    const fs_pitch<BIG> ldx2 = (fs_pitch<BIG>)ldx * 2, ldy2 = (fs_pitch<BIG>)ldy * 2;  // bytes between rows

    // descriptors of the unit's blocks (at most 64), one per lane
    const int4 my_desc = blk_desc[first + min(lane, nblk - 1)];

    for (int b0 = 0; b0 < nblk; b0 += BB) {
        // round of up to BB blocks: first every block's indices, row occupancies and X rows, then every Y row,
        // so that a round costs two memory round trips however many blocks it holds
        BlockDesc dsc[BB];
        int col[BB];
        uint32_t bits[BB];
        int rbase[BB];  // CSR position of window row j's first entry in the block (CSR-order output only)
        fs_frag xf[BB];
#pragma unroll
        for (int u = 0; u < BB; u++) {
            dsc[u] = fs_item_block(my_desc, b0 + u, nblk);
            col[u] = (lane < dsc[u].kb) ? vec_col[dsc[u].s + lane] : -1;
            bits[u] = row_bits[(int64_t)(first + min(b0 + u, nblk - 1)) * V + (j & (V - 1))];
            rbase[u] = 0;
            if constexpr (CSR) rbase[u] = (j < V && b0 + u < nblk) ? row_base[(int64_t)(first + b0 + u) * V + j] : 0;
            // X operand: lane (j, g) holds X[w*V + j][8g .. 8g+7]; rows past V or M are zero
            const int64_t xrow = (int64_t)dsc[u].w * V + j;
            const bool x_ok = dsc[u].kb > 0 && j < V && xrow < M;
            const uint64_t xoff = BIG ? (uint64_t)xrow * ldx2 : (uint64_t)fs_mul24((uint32_t)xrow, ldx2);
            xf[u].u = fs_u4{0u, 0u, 0u, 0u};
            if (x_ok && 8 * g < d) xf[u].u = *reinterpret_cast<const fs_u4 *>(Xb + xoff + 16 * g);
        }
        // Y operand: matrix row j of tile t is vector 8*(j/4) + 4t + (j%4) of the block; vectors past the
        // block's width re-read its first row and are masked out below
        fs_frag yf[BB][2];
#pragma unroll
        for (int u = 0; u < BB; u++) {
            const int first = max(__builtin_amdgcn_readfirstlane(col[u]), 0);
#pragma unroll
            for (int t = 0; t < 2; t++) {
                int yrow = __shfl(col[u], 8 * (j >> 2) + 4 * t + (j & 3), 64);
                yrow = yrow < 0 ? first : yrow;
                const uint64_t yoff = BIG ? (uint64_t)yrow * ldy2 : (uint64_t)fs_mul24((uint32_t)yrow, ldy2);
                yf[u][t].u = *reinterpret_cast<const fs_u4 *>(Yb + yoff + (8 * g < d ? 16 * g : 0));
                if (8 * g >= d) yf[u][t].u = fs_u4{0u, 0u, 0u, 0u};
            }
        }
#pragma unroll
        for (int u = 0; u < BB; u++) {
            const int kb = dsc[u].kb;
            if (kb <= 0) continue;
            fs_f4 acc[2];
#pragma unroll
            for (int t = 0; t < 2; t++) acc[t] = fs_mfma_16x16x32<DT>(yf[u][t], xf[u], fs_f4{0.f, 0.f, 0.f, 0.f});
            fs_store_scores<DT, V, CSR>(acc, bits[u], kb, rbase[u], lane, lds, out ? out + (int64_t)V * dsc[u].s : nullptr, out_csr);
        }
    }
}

template <int DT, int V>
fs_status launch(const fs_format *f, const uint16_t *X, int64_t ldx, const uint16_t *Y, int64_t ldy, int64_t d,
                 uint16_t *out, uint16_t *out_csr, hipStream_t st)
{
    if (f->n_blocks == 0) return FS_OK;
    const int n_blocks = (int)f->n_blocks;
    // The launch order pays where parts of hub windows are a good share of the items, what is read of Y is more than
    // one XCD's L2 holds, and there are wavefronts enough, because each then takes a whole item.  In order, us against
    // slot by slot, d = 128: R-MAT of 262 k rows, 17.5 k items, 75 and 108; of 65 k rows, 5.2 k items, 20 and 22; of
    // 32 k rows, 2.7 k items, 17 and 12; of 8 k rows, 0.6 k items, 9 and 5.  Items that are nearly all parts of hubs are
    // alike and get by with fewer (64 rows of 20 k entries among 4 k short ones, 1.8 k items: 12 and 18; 100 rows of
    // 5 k, 1.2 k items: 12 and 13, at d = 64 9 and 7).  For d <= 32 the rows are short and the L2s set the time:
    // only where hubs hold most of the work (500 rows of 4 k entries among 30 k short ones: 22 and 25; R-MAT of 131 k
    // rows: 21 and 20).
    const int64_t n_cut = f->n_cut_items, n_items = f->n_items;
    const bool ordered = fs_sddmm_in_order(f, d);
    // Otherwise up to four block slots per wavefront (4 to 8 measured best from 11 thousand to 200 thousand blocks, 16 and
    // more lose 5-15 %), fewer where that leaves less than eight wavefronts per CU: then a wavefront's own chain of steps
    // is the whole time (R-MAT of 8 k rows, 3 k blocks, d = 248: 14.1 us with four slots, 8.5 us with one).
    const int4 *items = ordered ? (const int4 *)f->items_by_cost : nullptr;
    int G = std::min(std::max(n_blocks / 2048, 1), 4);
    if (n_blocks >= 1 << 27) G = 16;  // (a launch has fewer than 2^32 threads)
#ifdef FS_TUNING_ENV  // tuning builds only (-DFS_TUNING_ENV): the shipped library reads no environment
    if (const char *e = getenv("FS_SDDMM_G")) G = std::min(std::max(atoi(e), 1), 64);
#endif
    // 32-bit row offsets need X and Y to span less than 4 GiB and row number and pitch to fit 24 bits
    const bool big = f->K >= ((int64_t)1 << 24) || f->M >= ((int64_t)1 << 24) || ldx * 2 >= ((int64_t)1 << 24) ||
                     ldy * 2 >= ((int64_t)1 << 24) || f->K * ldy * 2 >= ((int64_t)1 << 32) ||
                     (f->M + 32) * ldx * 2 >= ((int64_t)1 << 32);
    const fs_launch_geometry geo = fs_launch_geometry_for(f, 1);
    // 128 < d <= 256: whole rows at a time, or chunks of 128 features.  Whole rows are fetched once, and keep a window's rows of X, by
    // half the wavefronts; so they gain where rows of Y miss the L2s and windows are tall, and lose where rows hit.  Chunks / whole rows,
    // us, d = 136, 168, 200, 256, blocks in brackets, "in order" in launch order:
    //   eight rows: lognormal graph of 262 k rows (171 k) 381 / 288, 462 / 340, 540 / 390, 480 / 409; of 20 k rows (14 k) 20 / 23, 25 / 23,
    //     32 / 26, 33 / 28; of 15 k rows (10 k) 16 / 18, 17 / 19, 19 / 21, 23 / 22; stencil 500^2 (31 k) 50 / 46, 64 / 49, 81 / 57, 80 / 72; 300^2
    //     (11 k) 22 / 25, 25 / 27, 31 / 30, 31 / 34: from fifty blocks a CU on.  R-MAT of 32 k rows, hubs out of order (15 k) 20 / 23, 20 / 24,
    //     22 / 24, 24 / 25: not.  In order, 512 k rows (276 k) 322 / 330, 361 / 322, 439 / 350, 494 / 406; 131 k (66 k) 68 / 76, 69 / 71,
    //     83 / 74, 93 / 76: below d = 200 only where Y is much more than all L2s hold.
    //   sixteen: lognormal 262 k 459 / 312, 565 / 366, 658 / 420, 573 / 441; uniform 60 k rows (11 k) 30 / 26, 36 / 29, 43 / 33, 40 / 35; R-MAT of 262 k
    //     rows, in order 166 / 155, 209 / 134, 264 / 150, 287 / 174; of 32 k, hubs out of order (13 k) 19 / 21, 21 / 22, 24 / 23, 28 / 24; of 65 k (27 k)
    //     37 / 36, 43 / 38, 53 / 40, 64 / 46.
    //   four: lognormal 262 k (197 k) 334 / 281, 396 / 326, 466 / 378, 424 / 389, but uniform 60 k rows (15 k) 25 / 28, 29 / 30, 34 / 33, 32 / 34; stencil
    //     500^2, blocks of 14 vectors 67 / 82, 69 / 83, 74 / 86, 84 / 89; R-MAT of 262 k rows, a tenth of the items hubs (165 k) 159 / 184,
    //     170 / 190, 199 / 204, 289 / 264; of 1 M rows (1.1 M) 1193 / 1240, 1336 / 1257, 1594 / 1403, 1862 / 1688.
    // Up to d = 160 the second chunk is little work, and only rows that mostly miss the L2s gain.
    const int64_t y_bytes = f->K * d * 2;
    const bool tall = V == 16 ? n_blocks >= 8192 && (ordered || d >= 200 || n_blocks >= 25600 || n_cut * 8 < n_items * 3)
                      : V == 8 ? n_blocks >= 12800 && (ordered ? d >= 200 || y_bytes >= ((int64_t)64 << 20) : n_cut * 4 < n_items)
                               : f->nvec >= 18 * f->n_blocks && n_blocks >= (n_cut * 16 < n_items ? 1 << 15 : d >= 240 ? 1 << 16 : 1 << 19);
    const bool wide = tall && (d > 160 || (!ordered && y_bytes > ((int64_t)8 << 20)));
    const dim3 grid(ordered ? (unsigned)geo.nbx : (unsigned)(((int64_t)n_blocks + G - 1) / G)), block(64);
#define FS_SDDMM_ARGS items, (int)f->n_items, geo.slice, geo.n_swz, n_blocks, G, (const int4 *)f->blk_desc, f->vec_col, f->blk_row_bits, (int)f->nvec, X, ldx, Y, ldy, (int)d, out, f->M, out_csr, f->blk_row_base
#define FS_SDDMM_LAUNCH(...)  /* the kernel and its first template arguments */                         \
    {                                                                                                     \
        if (out_csr) {                                                                                    \
            if (big) __VA_ARGS__, true, true><<<grid, block, 0, st>>>(FS_SDDMM_ARGS);                     \
            else __VA_ARGS__, false, true><<<grid, block, 0, st>>>(FS_SDDMM_ARGS);                        \
        } else {                                                                                          \
            if (big) __VA_ARGS__, true, false><<<grid, block, 0, st>>>(FS_SDDMM_ARGS);                    \
            else __VA_ARGS__, false, false><<<grid, block, 0, st>>>(FS_SDDMM_ARGS);                       \
        }                                                                                                 \
    }
    if (d <= 32) FS_SDDMM_LAUNCH(k_sddmm_short<DT, V)
    else if (d <= 64) FS_SDDMM_LAUNCH(k_sddmm<DT, V, 2, 2, false)
    else if (d <= 128) FS_SDDMM_LAUNCH(k_sddmm<DT, V, 4, 1, false)
    else if (d <= 256 && wide) FS_SDDMM_LAUNCH(k_sddmm<DT, V, 8, 1, false)
    else FS_SDDMM_LAUNCH(k_sddmm<DT, V, 4, 1, true)
#undef FS_SDDMM_LAUNCH
#undef FS_SDDMM_ARGS
    FS_LAUNCH_CHECK();
    return FS_OK;
}

}  // namespace

fs_status fs_sddmm_launch(const fs_format *f, const void *d_X, int64_t ldx, const void *d_Y, int64_t ldy, int64_t d,
                          void *d_out_blk, void *d_out_csr, hipStream_t st)
{
    const uint16_t *X = (const uint16_t *)d_X, *Y = (const uint16_t *)d_Y;
    uint16_t *out = (uint16_t *)d_out_blk, *out_csr = (uint16_t *)d_out_csr;
    if (f->dtype == FS_F16) {
        if (f->V == 4) return launch<FS_F16, 4>(f, X, ldx, Y, ldy, d, out, out_csr, st);
        if (f->V == 8) return launch<FS_F16, 8>(f, X, ldx, Y, ldy, d, out, out_csr, st);
        if (f->V == 16) return launch<FS_F16, 16>(f, X, ldx, Y, ldy, d, out, out_csr, st);
    } else if (f->dtype == FS_BF16) {
        if (f->V == 4) return launch<FS_BF16, 4>(f, X, ldx, Y, ldy, d, out, out_csr, st);
        if (f->V == 8) return launch<FS_BF16, 8>(f, X, ldx, Y, ldy, d, out, out_csr, st);
        if (f->V == 16) return launch<FS_BF16, 16>(f, X, ldx, Y, ldy, d, out, out_csr, st);
    }
    return FS_ERR_UNSUPPORTED;
}
