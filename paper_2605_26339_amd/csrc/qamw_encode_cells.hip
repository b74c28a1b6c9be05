// QAM-W encoder with a cell table made on the device (Sec. 3.1 / Sec. 3.5; the index is the one the search over the
// whole codebook returns, lowest index on ties).
//
// k_cells_prepare cuts a square that follows the codebook's scale into G x G cells and lists, per cell, every codeword that can
// be nearest to a point of the cell; the same launch computes the row norms that the search does not.  k_encode_cells keeps the codebook and the whole table
// in LDS and decides a pair by the exact fp32 squared distances to its cell's first four candidates, and to the fifth where there
// is one (0.14 % of the pairs that a Lloyd codebook of 2^11 points is for).  A pair outside the table (0.0002 % of them), or in a
// cell that lists more (0.001 %), is decided by the exact scan of the whole codebook (64 lanes x K/64 codewords).
//   Where that meets many of an item's pairs -- pairs much wider than the codebook, codewords that no Lloyd iteration has spread
// -- the item is put off: once the wave has walked its rows it takes those without the table, all 512 pairs together
// (nearest_of_all(); all distances up to 32 codewords).  That loop comes after the other and not inside it so that it costs
// the other no registers.  After an item was put off the next is too, then the next 3, 7, 15, without a try.
//
// What bounds k_encode_cells: the issue of its instructions (606 of the vector ALU, 140 scalar and 42 of LDS for a wave's 512
// pairs), with four waves per SIMD to hide the LDS gathers behind.  A SIMD issues a vector instruction in 2.1 cycles, but one in
// four of the kind that min, max, compare, shift and DPP are (adds, multiplies, ANDs and moves go in between), so what helps is
// fewer instructions, and waves that do not wait at the same time.  Hence one workgroup of 16 waves per CU that stages its 144 KB
// once and walks the rows; a wave keeps to one 1024-column slab of a matrix, so the slab's scales, signs and pair gains are
// loaded, divided and combined once per wave instead of once per row; records of all eight pairs requested at once, and a pair's
// candidates before the pair ahead of it is decided.  13824 x 5120 at 11 bits, the whole call: 134 us with five candidates in cells
// of one width, a comparison and two selections each, so 98 (a 7B layer with the pair scales 398, so 313; of both 1.1 by the order of the
// waves, see below).
//   Row norms.  Of large matrices whose rows have 2, 4 or 8 slabs (see cells_shares_rows()) they are computed here (OWN): a row's waves are
// neighbours in a workgroup, and each sums the slab of its next row, which is in its registers anyway, while the present one is searched, so that
// the matrix is read from memory once.  The launch ahead of this then makes the table and the other norms: a 7B layer's 82 -> 22 us by
// the trace, this one 187 -> 220 (7 of them the sums, 12 the waits for a row's other waves); the call 313 -> 290.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "qamw_cells.hpp"

namespace qamw {

// Launches at 2^11 points of at most this many (row, slab) items read the records from memory.  In us a call, from LDS / from
// memory (bf16): 256 x 2048, 512 items, 27.0 / 23.6; 1500 x 2048, 3000 items, 28.1 / 26.4; 2048 x 2048, 4096 items, 30.8 / 30.0;
// 1024 x 8192, 8192 items, 36.0 / 37.5; 4096 x 4096 48.5 / 52.1.  The smaller tables (32 to 72 KB) are staged in less than the
// second L2 round trip takes: 1024 x 2048 at 10 bits 20.3 / 19.6, at 7 bits 18.7 / 25.1.
constexpr int CELLS_DIRECT_MAX_ITEMS = 3072;
constexpr int CELLS_ROWS_TOGETHER = 8192;                      // rows of a launch from which a wave sums four
// Where the encoder computes row norms itself: matrices whose rows a workgroup's waves share without many idle lanes, and enough of
// them, for that costs its waves more instructions, and waits for a row's other waves, than a second reading from memory does beside
// the making of the table.  us a call, norms in the first launch / in the encoder, bf16: 4 slabs 8192 x 4096 (64 MiB) 50 / 51, 10240 55.6 /
// 56.1, 12288 65.3 / 63.8, 14336 73.4 / 72.1, at 10 bits 74 / 68.5; 2 slabs 16384 x 2048 51.6 / 49.2, 22016 65.7 / 61.5; 8 slabs 4096 x 8192 46.9 / 50.2,
// 7168 72.1 / 75.2, 8192 (128 MiB) 88 / 84, 28672 289 / 257; one slab 32768 x 1024 46.4 / 49.4, 65536 78.7 / 79.1; 16 slabs 4096 x 16384 80 / 102;
// last slabs not full 17387 x 3136 76.6 / 80, 19660 x 3840 90.3 / 91.3, 9830 x 7680 90.8 / 95.4, 49152 x 1536 100 / 105.  fp32, whose norms in the
// first launch read twice as much: 4096 x 4096 (64 MiB) 36.3 / 36.7, 6144 46.0 / 43.5, 8192 64.6 / 51.3; 20480 x 1024 41.7 / 39.9; 4096 x 8192 56.1 / 51.8;
// 12288 x 1536 40.8 / 40.7.  Last slabs that are not full are out in fp32 too: their waves have fewer undecided pairs than the others that they
// wait for, and which way the workgroup goes suits only some (12288 x 1536 at 7 bits, pairs 2.5 times as wide as the codebook: 205 / 326).
//   A 7B layer (315 MB in rows of 4 slabs, 90 in rows of 11) 313 / 290 with the pair scales.
constexpr int CELLS_OWN_MOST_SLABS = 8;
constexpr bool cells_shares_rows(int dtype, int n_slabs, int d_in) {
    return CELLS_OWN_MOST_SLABS % n_slabs == 0 && d_in == 1024 * n_slabs && (n_slabs > 1 || dtype == 0);
}
// 64 MiB of matrices of one or two slabs, 96 of four, 128 of eight, or parts of each.
constexpr int64_t CELLS_OWN_MIN_BYTES = 32 << 20;
constexpr int cells_own_parts(int log_slabs) { return log_slabs < 1 ? 2 : 1 + log_slabs; }
constexpr int CELLS_MIN_ITEMS = 4096;                          // (row, slab) items of a launch from which small codebooks use the table,
constexpr int CELLS_GRID_MIN_ITEMS = 1024;                     // and from which the pruned search does

struct CellsMat {
    const void *W;
    int64_t ldw;
    const float *chan_scale;
    const int8_t *signs;
    const float *pair_sigma;
    float *norms;
    uint8_t *packed;
    int64_t row_bytes;
    int d_in, d_out, n_slabs, slab_sums;
    int own_norms, log_slabs;                    // the encoder computes the norms: 2^log_slabs waves of a workgroup share a row
    float g_default;
};
struct CellsBatch {
    CellsMat m[QAMW_ENCODE_MAX_BATCH];
    int norm_begin[QAMW_ENCODE_MAX_BATCH + 1];   // k_cells_prepare: first norm workgroup of each matrix
    int n, bits, K;
    float inv_sqrt_block, half_per_sum;
    int dense_above;                             // with more undecided pairs than this all pairs of an item are searched anew
    int grid_side;
    const uint32_t *grid;                        // the caller's table (qamw_search_grid_build), nullable
    const float *codebook;
    uint2 *table;                                // G x G records
};

// ------------------------------------------------------------------------------------------------ table and norms
// Workgroups 0 .. (G/8)^2 - 1 make the table; the rest compute the row norms that the encoder does not.
// R rows per wave: large launches take four, which fetches the channel scales (twice the bytes of bf16 weights) a quarter as
// often.  A 7B layer, 405 MB: 87 us with one row per wave, 77 so (84 with the sums slab by slab;
// by the trace 86 us, 79 since a square is added in one operation and four rows share the last steps of their butterflies).
template <int DTYPE, int G, int R>
__global__ __launch_bounds__(CP_THREADS) void k_cells_prepare(CellsBatch bt) {
    constexpr int REGIONS = (G / 8) * (G / 8);
    if (blockIdx.x < REGIONS) {
        const float2 *codebook = reinterpret_cast<const float2 *>(bt.codebook);
        cells_build_region<G>(cells_points(bt.K, [=](int i) { return codebook[i]; }), bt.K, bt.half_per_sum, bt.table, (int)blockIdx.x);
        return;
    }
    const int b = (int)blockIdx.x - REGIONS;
    int mi = 0;
    while (mi + 1 < bt.n && b >= bt.norm_begin[mi + 1]) ++mi;
    const CellsMat &M = bt.m[mi];
    const int lane = threadIdx.x & (WAVE - 1);
    const int row = __builtin_amdgcn_readfirstlane(((b - bt.norm_begin[mi]) * CP_WAVES + (int)(threadIdx.x >> 6)) * R);
    if (row >= M.d_out) return;
    const int n_rows = min(R, M.d_out - row);
    if (M.slab_sums) {
        const double s2 = wave_rows_slab_sums<DTYPE, R>(M.W, row, n_rows, M.ldw, M.d_in, M.chan_scale, lane);
        const int r = lane / (WAVE / R);
        if (lane % (WAVE / R) == 0 && r < n_rows) M.norms[row + r] = (float)sqrt(s2);
        return;
    }
    double s2[R];
    wave_rows_sum_of_squares<DTYPE, R>(s2, M.W, row, n_rows, M.ldw, M.d_in, M.chan_scale, lane);
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r < n_rows) M.norms[row + r] = (float)sqrt(s2[r]);
    }
}

// ------------------------------------------------------------------------------------------------ the encoder
constexpr int CELLS_DIRECT_THREADS = 256;
constexpr int cells_threads(int G, bool own) { return G == 128 || (G == 96 && own) ? 1024 : 512; }
constexpr int cells_codewords(int G) { return G == 128 ? 2048 : G == 96 ? 1024 : 512; }
constexpr int cells_least_k(int G) { return G == 128 ? 2048 : G == 96 ? 1024 : 2; }
constexpr int cells_bits(int G) { return G == 128 ? 11 : G == 96 ? 10 : 0; }   // 0: 1 to 9
// How many rows the workgroup's waves have taken: in the lower word of a corner's record, which has no candidates (whatever is there,
// the reads that it makes end below 16 KB and are not looked at).
constexpr uint32_t cells_count_at(int G) { return (uint32_t)(cells_codewords(G) * 8 + (G - 1) * 8); }
// In the two others that hold nothing else, where the encoder computes norms: the undecided pairs of the workgroup's recent items, and
// whether items are put off; see cells_many().
constexpr uint32_t cells_level_at(int G) { return (uint32_t)(cells_codewords(G) * 8 + (G * G - 1) * 8); }
constexpr uint32_t cells_puts_at(int G) { return (uint32_t)(cells_codewords(G) * 8 + (G * G - G) * 8); }
// Norms that the encoder computes: after codebook and table the slab sums of the waves' next rows, then per group of waves that share
// rows (groups of 16 / n from number n on) how many are there, then the norm and of which row it is.
constexpr int CELLS_GROUPS = 32;
constexpr uint32_t cells_part_at(int G) { return (uint32_t)(cells_codewords(G) * 8 + G * G * 8); }
constexpr uint32_t cells_arrived_at(int G) { return cells_part_at(G) + 16 * 8; }
constexpr uint32_t cells_norm_at(int G) { return cells_arrived_at(G) + CELLS_GROUPS * 4; }
constexpr size_t cells_lds_bytes(int G, bool own) { return own ? cells_norm_at(G) + CELLS_GROUPS * 8 : cells_part_at(G); }
// Workgroups that a CU holds.  Codebook and table of 10 bits are half of its LDS to the byte, so with norms there is one of 16 waves
// (with one of 8, and the launch's others after it, 11008 x 4096 bf16 took 82 us, 13824 x 5120 without norms 102; so 64 and 87; two
// of 8 and the norms from the launch ahead 65, but a 7B layer 263 instead of 225, in fp32 402 instead of 290.  Small launches have
// more workgroups of 8 waves: 512 x 4096 16.2, with those of 16 17.5).
//   With fp32 weights 8 waves' registers (130 to 177 a lane) leave no room for 8 more.  Twice as many workgroups, the second half
// after the first, each with a table to stage: 1024 x 4096 at 7 bits 18.7 us, 15.6 so, at 10 bits 20.9, 17.2; 4096 x 4096 at 7 bits 38.9, 35.7.
constexpr int cells_per_cu(int G, bool own, int dtype) { return cells_threads(G, own) == 1024 || dtype == 0 ? 1 : 2; }
template <int G, bool OWN> constexpr bool cells_resident(int dtype) { return cells_per_cu(G, OWN, dtype) * cells_lds_bytes(G, OWN) <= 160 * 1024; }

// The constants of a lane's 16 columns from c on: scale x sign per column, gain per pair.  True: see combine_gains().
template <int B>
__device__ __forceinline__ bool cells_constants(float (&sc)[16], float (&g)[8], const CellsMat &M, int c, float parity, float inv_sqrt_block) {
    Problem p;
    p.chan_scale = M.chan_scale;
    p.signs = M.signs;
    p.pair_sigma = M.pair_sigma;
    p.g_default = M.g_default;
    load_signed_scales(sc, p, c);
    load_pair_gains(g, p, c);
    return unit_exact(B) && combine_gains(g, parity, inv_sqrt_block);
}
// A lane's pairs from its raw words: rotated_unit_row with the sign folded into the scale (exact).
template <int DTYPE, int B>
__device__ __forceinline__ void cells_pairs(float (&x)[16], const RawRow<DTYPE> &raw, float norm, const float (&sc)[16], const float (&g)[8],
                                            const LaneSigns<B> &ls, float unit, bool two, float inv_sqrt_block) {
    widen_raw_row<DTYPE>(x, raw);
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = x[e] * sc[e];
    divide_by_norm(x, norm);
    fwht_wave<B>(x, ls);
    if (unit_exact(B) && __builtin_expect(two, false)) {
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = x[e] * inv_sqrt_block;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = (unit_exact(B) ? x[e] : x[e] * unit) * g[e >> 1];
}

// The waves of the launch take the (row, slab) items of a matrix in turn, `step` at a time, a multiple of the slab count: a
// wave stays on its slab.  The next matrix begins with the wave after the last one that got an item.
struct CellsShare {
    int row, rows_step, slab;                                  // the wave's rows of the matrix: row, row + rows_step, ... of one slab
};
// False: the wave has no item of M.  gw: the wave's number; turn: the wave that takes M's first item, on return the next matrix's.
__device__ __forceinline__ bool cells_share(CellsShare &out, const CellsMat &M, int gw, int n_waves, int &turn) {
    const int n_slabs = M.n_slabs, n_items = M.d_out * n_slabs;
    const int rows_step = n_waves / n_slabs, step = rows_step * n_slabs;
    if (M.own_norms) {                                         // a row's waves in one workgroup
        turn = (turn + n_slabs - 1) & -n_slabs;                // a power of two
        if (turn >= n_waves) turn -= n_waves;
    }
    int local = gw - turn;
    if (local < 0) local += n_waves;
    turn += n_items % step;
    if (turn >= n_waves) turn -= n_waves;
    if (local >= step || local >= n_items) return false;
    out.row = local / n_slabs;
    out.slab = local - out.row * n_slabs;
    out.rows_step = rows_step;
    return true;
}
constexpr int cells_together(int G, int B) { return G == 64 && B <= 256 ? 4 : 2; }   // pairs of a lane that nearest_of_all() takes: what the registers hold
constexpr int CELLS_FEW_LANES = 12;                            // lanes with an undecided pair: up to here their pairs are scanned one by one
constexpr int CELLS_PUT_OFF = 256;                             // items of a wave that can be put off, a bit each (in scalar registers)

// Whether an item with n_scan undecided pairs, in more than a few lanes, is put off.  A little before the line, since waves finish late
// that have some items of either kind by chance.  Where a row's waves wait for each other to have its norm they go one way: with some items
// put off and some scanned all waited for those that scan, and the others gained nothing (12288 x 4096 bf16, 2048 points, pairs 2.8
// times as wide as the codebook, the line at 57: 2320 us; all scanned 1295, none 2010).  So there a wave's first such item is put off
// sooner, and then the mean over the workgroup's recent ones counts: the workgroup keeps its way until that is an eighth beyond the
// line, and only an item far from it goes its own.  (Of waves that come here together each counts as if it were alone, which is near enough.)
constexpr int CELLS_LEVEL_UNIT = 64, CELLS_LEVEL_FIRST = 16, CELLS_LEVEL_ITEMS = 32;
constexpr uint32_t CELLS_NO_WAY = 2;                            // so far
template <int G, bool OWN> __device__ __forceinline__ bool cells_many(int n_scan, int dense_above, bool first, int lane) {
    if (!OWN) return 16 * n_scan > 13 * dense_above;
    const int line = CELLS_LEVEL_UNIT * 15 / 16 * dense_above;
    const uint32_t puts = __builtin_amdgcn_readfirstlane(lds_read<uint32_t>(cells_puts_at(G)));
    int level = __builtin_amdgcn_readfirstlane((int)lds_read<uint32_t>(cells_level_at(G)));
    const int step = (CELLS_LEVEL_UNIT * n_scan - level) / (puts == CELLS_NO_WAY ? CELLS_LEVEL_FIRST : CELLS_LEVEL_ITEMS);
    if (lane == 0) lds_add(cells_level_at(G), (uint32_t)step);
    level += step;
    uint32_t now = puts;
    if (puts == CELLS_NO_WAY ? !first : level > line + line / 8 || level < line - line / 8) now = level > line ? 1u : 0u;
    if (now != puts && lane == 0) lds_write<uint32_t>(cells_puts_at(G), now);
    if (first && puts == CELLS_NO_WAY) return 16 * n_scan > 11 * dense_above;
    return n_scan > 2 * dense_above || (2 * n_scan > dense_above && now);
}

// Registers: 16 waves per CU, of one workgroup or two; with fp32 weights and tables below 128 x 128 that would cost spills, and there are 8.
#define QAMW_CELLS_WAVES_PER_EU ((STAGED && (cells_threads(G, OWN) == 1024 || DTYPE == 1)) ? 4 : 2)
// STAGED: the table in LDS beside the codebook.  Otherwise its records are read from memory (L2): in a launch of few items a
// workgroup would stage 128 KB for an item or two per wave, and small workgroups reach more CUs.
template <int DTYPE, int B, int G, bool STAGED, bool OWN>
__global__ __launch_bounds__(STAGED ? cells_threads(G, OWN) : CELLS_DIRECT_THREADS) __attribute__((amdgpu_waves_per_eu(QAMW_CELLS_WAVES_PER_EU)))
void k_encode_cells(CellsBatch bt) {
    static_assert(STAGED || (G & (G - 1)) == 0, "the mask of the record's offset");
    static_assert(STAGED || !OWN, "the sums' place in LDS is after the table's");
    static_assert(!STAGED || cells_resident<G, OWN>(DTYPE), "the launch's workgroups are resident together");
    constexpr int THREADS = STAGED ? cells_threads(G, OWN) : CELLS_DIRECT_THREADS, WAVES = THREADS / WAVE;
    constexpr int CODEWORDS = cells_codewords(G);
    constexpr uint32_t TABLE_AT = CODEWORDS * 8;               // LDS: the codebook at 0, then the table
    const int K = cells_bits(G) ? CODEWORDS : bt.K, bits = cells_bits(G) ? cells_bits(G) : bt.bits;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LaneSigns<B> ls(lane);
    // The lane's first column in a slab.  (Of fp32 kernels with 128 x 128 cells every register counts: with the position kept too, 18 to 20
    // were spilled, and scratch memory is what short launches pay for.  1024 x 4096 22.4 us, 18.4 so; 4096 x 2048 29.9, 25.4.)
    const int lane_col = 16 * slab_pos(lane);
    const float unit = ls.parity * bt.inv_sqrt_block;
    const int n_waves = (int)gridDim.x * WAVES;
    const int gw = (int)blockIdx.x * WAVES + wid;

    // The wave's items, matrix by matrix, one slab of each.  The next row -- the next matrix's first after the last one of this --
    // is on its way while one is searched: a wave meets a matrix every four to eleven rows of a 7B layer, and waited there for memory
    // as all others did.
    int mi = -1, turn = 0;                                      // the matrix that the next row is of
    CellsShare share;
    const char *w_next = nullptr;                               // the wave's next row
    float *norm_at = nullptr;
    int64_t w_step = 0;
    int left = 0;                                               // rows of it that the wave has yet to ask for
    auto next_matrix = [&]() __attribute__((always_inline)) {
        while (++mi < bt.n) {
            const CellsMat &M = bt.m[mi];
            if (!cells_share(share, M, gw, n_waves, turn)) continue;
            const int64_t pitch = M.ldw * (DTYPE == 0 ? 4 : 2);
            w_next = static_cast<const char *>(M.W) + share.row * pitch;
            w_step = share.rows_step * pitch;
            norm_at = M.norms + share.row;
            left = (M.d_out - share.row + share.rows_step - 1) / share.rows_step;
            return;
        }
    };
    RawRow<DTYPE> next;
    float norm_next = 0.0f;
    uint32_t tag_next = 0;                                      // not 0: the next row's norm is this launch's, the row's mark
    float *norm_out = nullptr;
    auto first_column = [&](int slab, int d_in) __attribute__((always_inline)) {
        const int col0 = slab * 1024 + lane_col;
        return col0 < d_in ? col0 : 0;
    };
    auto request = [&]() __attribute__((always_inline)) {       // the next row
        if (left == 0) next_matrix();
        tag_next = 0;
        if (mi >= bt.n) return;
        load_raw_row<DTYPE>(next, w_next, 0, first_column(share.slab, bt.m[mi].d_in));
        w_next += w_step;
        --left;
        if (OWN && bt.m[mi].own_norms) {
            tag_next = (uint32_t)(mi + 1) << 24 | (uint32_t)left;   // fewer than 2^24: see the launch
            norm_out = norm_at;
        } else {
            norm_next = *norm_at;
        }
        norm_at += share.rows_step;
    };
    request();

    // the codebook and the table, requested in one go
    const float half = cells_half(bt.table);
    {
        constexpr int CB = (CODEWORDS + THREADS - 1) / THREADS, RECS = STAGED ? (G * G / 2 + THREADS - 1) / THREADS : 0;
        constexpr bool WHOLE = G * G / 2 % THREADS == 0;
        const lds_f32x2_t *cbk = reinterpret_cast<const lds_f32x2_t *>(bt.codebook);
        const lds_u32x4_t *src = reinterpret_cast<const lds_u32x4_t *>(bt.table);
        lds_f32x2_t c[CB];
        lds_u32x4_t r[RECS + 1];
#pragma unroll
        for (int i = 0; i < CB; ++i) c[i] = cbk[min((int)threadIdx.x + i * THREADS, K - 1)];
#pragma unroll
        for (int i = 0; i < RECS; ++i) r[i] = src[WHOLE ? (int)threadIdx.x + i * THREADS : min((int)threadIdx.x + i * THREADS, G * G / 2 - 1)];
#pragma unroll
        for (int i = 0; i < CB; ++i)
            if (cells_bits(G) || (int)threadIdx.x + i * THREADS < K) lds_write(8 * (threadIdx.x + i * THREADS), c[i]);
#pragma unroll
        for (int i = 0; i < RECS; ++i)
            if (WHOLE || (int)threadIdx.x + i * THREADS < G * G / 2) lds_write(TABLE_AT + 16 * (threadIdx.x + i * THREADS), r[i]);
    }
    asm volatile("" ::: "memory");                             // (the threads that have written those records)
    if (STAGED && threadIdx.x == (G - 1) / 2) lds_write<uint32_t>(cells_count_at(G), 0u);
    if (OWN && threadIdx.x == (G * G / 2 - G / 2) % THREADS) lds_write<uint32_t>(cells_puts_at(G), CELLS_NO_WAY);
    if (OWN && threadIdx.x == (G * G / 2 - 1) % THREADS) lds_write<uint32_t>(cells_level_at(G), (uint32_t)(CELLS_LEVEL_UNIT * bt.dense_above));
    if (OWN && threadIdx.x < 3 * CELLS_GROUPS) lds_write<uint32_t>(cells_arrived_at(G) + 4 * threadIdx.x, 0u);
    __syncthreads();

    float sc[16], g[8];
    // The sum of squares of the wave's slab of its next row, and the row's norm if the row's other waves have left theirs.  In the order
    // of the kernels without scratch (a sign is nothing to a square, and wave_sum() meets the same pairs in slab_pos()'s order).
    //   A wave's place for its sum, and its group's for the norm, are free by then: the wave has had the norm of the row that it works
    // on, so that row's sums are read, and a norm follows only when all waves of the group have come as far.
    auto sum_next = [&](int now) __attribute__((always_inline)) {
        const CellsMat &M = bt.m[mi];
        const int col0 = share.slab * 1024 + lane_col;
        if (mi != now) {                                        // the row is another matrix's: this one's scales are done with
            Problem p;
            p.chan_scale = M.chan_scale;
            p.signs = nullptr;
            load_signed_scales(sc, p, col0 < M.d_in ? col0 : 0);
        }
        float w[16];
        widen_raw_row<DTYPE>(w, next);
        double s2 = 0.0;
#pragma unroll
        for (int e = 0; e < 16; ++e) s2 = add_square(s2, w[e] * sc[e]);
        s2 = wave_sum(col0 < M.d_in ? s2 : 0.0);
        const int log = M.log_slabs, first = wid >> log << log, id = (16 + wid) >> log;
        uint32_t before = 0;
        if (lane == 0) {
            lds_write<double>(cells_part_at(G) + 8 * wid, s2);
            asm volatile("" ::: "memory");                      // before the arrival (LDS takes a wave's accesses in order)
            before = lds_add(cells_arrived_at(G) + 4 * id, 1u);
        }
        if ((int)__builtin_amdgcn_readfirstlane(before) != (1 << log) - 1) return;
        asm volatile("" ::: "memory");
        double sum = 0.0;                                       // in slab order
        for (int i = 0; i < 1 << log; ++i) sum += lds_read<double>(cells_part_at(G) + 8 * (first + i));
        const float norm = (float)sqrt(sum);
        if (lane == 0) {
            lds_write<uint32_t>(cells_arrived_at(G) + 4 * id, 0u);
            asm volatile("" ::: "memory");                      // before the norm, after which the next arrivals come
            lds_write<lds_u32x2_t>(cells_norm_at(G) + 8 * id, lds_u32x2_t{__float_as_uint(norm), tag_next});
            *norm_out = norm;
        }
    };
    // The norm of the row marked `tag`.  The wait ends: the row's other waves, all of this workgroup, leave their sums with the row
    // before it, for which they wait only for sums left with the row before that, and so on to the first, which they wait for none with.
    auto wait_for_norm = [&](int log, uint32_t tag) __attribute__((always_inline)) {
        const auto *at = reinterpret_cast<const volatile __attribute__((address_space(3))) uint64_t *>(cells_norm_at(G) + 8 * ((16 + wid) >> log));
        for (;;) {
            const uint64_t v = *at;
            if ((uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) == tag) return __uint_as_float((uint32_t)v);
            __builtin_amdgcn_s_sleep(1);
        }
    };
    if (OWN && tag_next) sum_next(-1);

    const float inv_span = cells_inv_span(half), far = cells_far(half);
    unsigned long long put_off[CELLS_PUT_OFF / 64] = {};        // items that the table does not help
    auto put = [&](int n) {
#pragma unroll
        for (int q = 0; q < CELLS_PUT_OFF / 64; ++q) put_off[q] |= n >> 6 == q ? 1ull << (n & 63) : 0ull;
    };
    bool any_put_off = false;
    int skip = 0, streak = 0;                                   // items still to be put off untried; how many at a time
    int n = 0;                                                  // the wave's items so far
#pragma unroll 1
    while (mi < bt.n) {
        const CellsMat &M = bt.m[mi];
        const int col0 = share.slab * 1024 + lane_col;
        const bool active = col0 < M.d_in;
        const int c = active ? col0 : 0;
        const unsigned long long lanes = __ballot(active);
        const int64_t row_bytes = M.row_bytes;
        const int d_in = M.d_in;
        uint8_t *out = M.packed + share.row * row_bytes;
        const int64_t out_step = share.rows_step * row_bytes;
        const int now = mi;
        const bool two = cells_constants<B>(sc, g, M, c, ls.parity, bt.inv_sqrt_block);

        for (int rows = left + 1; rows > 0; --rows, ++n, out += out_step) {
            const RawRow<DTYPE> raw = next;
            float norm = norm_next;
            const uint32_t tag = tag_next;
            request();
            if (OWN && tag) norm = wait_for_norm(M.log_slabs, tag);
            // Four waves share a SIMD, and the oldest goes first: the others finished up to half as late again, alone on their SIMD
            // by then.  So a wave that is behind the workgroup's average goes before one that is not.
            unsigned done = 0;                                  // by the workgroup
            if (STAGED && lane == 0) done = lds_add(cells_count_at(G), 1u);
            const bool try_table = skip == 0 || n >= CELLS_PUT_OFF;
            float x[16];
            if (try_table) {
                if constexpr (STAGED && G == 128 && DTYPE == 0) {   // no registers for the lane's signs: made again
                    int col = lane_col;
                    asm volatile("" : "+v"(col));
                    cells_pairs<DTYPE, B>(x, raw, norm, sc, g, LaneSigns<B>(lane, col >> 4), unit, two, bt.inv_sqrt_block);
                } else {
                    cells_pairs<DTYPE, B>(x, raw, norm, sc, g, ls, unit, two, bt.inv_sqrt_block);
                }
            }
            if (OWN && tag_next) sum_next(now);              // by now the next row has come
            if (!try_table) {
                --skip;
                put(n);
                continue;
            }

            // ---------------- the cells' records
            uint2 rec[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t at = cells_record_at<G>(x[2 * k], x[2 * k + 1], inv_span, STAGED ? TABLE_AT : 0u);
                if (STAGED) {
                    const lds_u32x2_t r = lds_read<lds_u32x2_t>(at);
                    rec[k] = make_uint2(r[0], r[1]);
                } else {
                    rec[k] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const char *>(bt.table) + (at & (G * G * 8u - 1u)));   // in range whatever x is
                }
            }
            // A pair's candidates are requested before the pair ahead of it is decided; otherwise a wave waits for LDS sixteen times.
            __builtin_amdgcn_sched_barrier(0);
            unsigned idx8[8];                                   // 8 times the index: the codeword's byte offset
            unsigned any = 0;
            CellsFour four[2];
            cells_request(four[0], rec[0], 0u);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k + 1 < 8) cells_request(four[(k + 1) & 1], rec[k + 1], 0u);
                __builtin_amdgcn_sched_barrier(0);
                any |= rec[k].y;
                idx8[k] = cells_offset(cells_nearest(four[k & 1], x[2 * k], x[2 * k + 1]));
                __builtin_amdgcn_sched_barrier(0);
            }

            // ---------------- the rest: fifth candidates, ...
            if (__ballot(any >= CELLS_SCAN || (any & CELLS_BORDER)) != 0ull) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (__ballot(rec[k].y & CELLS_FIFTH) == 0ull) continue;
                    const lds_f32x2_t cw = lds_read<lds_f32x2_t>(idx8[k]);
                    const double best = cells_candidate(exact_dist2(x[2 * k], x[2 * k + 1], make_float2(cw[0], cw[1])), idx8[k]);
                    idx8[k] = cells_offset(cells_fifth(rec[k], x[2 * k], x[2 * k + 1], 0u, best));
                }
                // ... and pairs that no record decides, a few by the exact scan, the whole wave on one pair at a time; many later
                if (__ballot(any & (CELLS_SCAN | CELLS_BORDER)) & lanes) {
                    unsigned long long scan[8], flagged = 0;    // lanes whose k-th pair is scanned
                    int n_scan = 0;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        scan[k] = __ballot(cells_undecided<false>(rec[k], x[2 * k], x[2 * k + 1], far)) & lanes;
                        flagged |= scan[k];
                        n_scan += __popcll(scan[k]);
                    }
                    // many: without the table, later.  (A grid decides most of them; otherwise as many as dense_above.)
                    if (__popcll(flagged) > CELLS_FEW_LANES && n < CELLS_PUT_OFF && (bt.grid || cells_many<G, OWN>(n_scan, bt.dense_above, !any_put_off, lane))) {
                        put(n);
                        if (!OWN || any_put_off || n_scan > 2 * bt.dense_above) skip = streak = min(2 * streak + 1, 15);
                        any_put_off = true;
                        continue;
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        unsigned long long mask = scan[k];
                        while (mask) {
                            const int src = __ffsll((long long)mask) - 1;
                            mask &= mask - 1;
                            const int bi = wave_exact_scan<cells_least_k(G), CODEWORDS>(lane_value(x[2 * k], src), lane_value(x[2 * k + 1], src), 0u, K, lane);
                            if (lane == src) idx8[k] = 8u * (unsigned)bi;
                        }
                    }
                }
            }
            streak = 0;
            if (STAGED) {
                if (__builtin_amdgcn_readfirstlane(done) < (unsigned)(n * WAVES)) __builtin_amdgcn_s_setprio(0);
                else __builtin_amdgcn_s_setprio(2);
            }

            int at = c;                                         // (the lane's place in a row is not worth registers during the search)
            asm volatile("" : "+v"(at));
            if (active) store_fields<3>(out, row_bytes, d_in, at, idx8, bits);
        }
    }
    if (OWN) __syncthreads();                                   // the norms are in memory
    if (!any_put_off) return;

    // ---------------- the items put off: all their pairs against the whole codebook.  All that follows from the lane is made
    // again: it is not worth registers during the search above.
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const LaneSigns<B> ls2(ln);
    const float unit2 = ls2.parity * bt.inv_sqrt_block;
    n = 0;
    turn = 0;
#pragma unroll 1
    for (int mi = 0; mi < bt.n; ++mi) {
        const CellsMat &M = bt.m[mi];
        if (!cells_share(share, M, gw, n_waves, turn)) continue;
        const int col0 = share.slab * 1024 + 16 * slab_pos(ln);
        const bool active = col0 < M.d_in;
        const int c = active ? col0 : 0;
        for (int row = share.row; row < M.d_out; row += share.rows_step, ++n) {
            unsigned long long bits64 = 0;
#pragma unroll
            for (int q = 0; q < CELLS_PUT_OFF / 64; ++q) bits64 = n >> 6 == q ? put_off[q] : bits64;
            if (!((bits64 >> (n & 63)) & 1ull)) continue;
            float x[16];
            {
                float sc[16], g[8];
                const bool two = cells_constants<B>(sc, g, M, c, ls2.parity, bt.inv_sqrt_block);
                RawRow<DTYPE> raw;
                load_raw_row<DTYPE>(raw, M.W, (int64_t)row * M.ldw, c);
                cells_pairs<DTYPE, B>(x, raw, M.norms[row], sc, g, ls2, unit2, two, bt.inv_sqrt_block);
            }
            unsigned idx8[8];
            bool decided = false;
            if (G == 64 && K <= 32) {                           // few codewords: all distances
                decided = true;
                float bd[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    bd[k] = 3.0e38f;
                    idx8[k] = 0;
                }
#pragma unroll 1
                for (uint32_t at = 0; at < 8u * (uint32_t)K; at += 8) {
                    const lds_f32x2_t cw = lds_read<lds_f32x2_t>(at);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const float dd = exact_dist2(x[2 * k], x[2 * k + 1], make_float2(cw[0], cw[1]));
                        idx8[k] = dd < bd[k] ? at : idx8[k];
                        bd[k] = fminf(bd[k], dd);
                    }
                }
            } else if (bt.grid) {                                      // the caller's table has smaller cells and eight candidates
                const uint4 *cells = reinterpret_cast<const uint4 *>(bt.grid + 8);
                const float grid_inv_h = __uint_as_float(bt.grid[4]);
                uint4 rec[8];
                unsigned scan = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    bool inside;
                    rec[k] = cells[grid_cell(x[2 * k], x[2 * k + 1], grid_inv_h, bt.grid_side, inside)];
                    if (!inside) scan |= 1u << k;
                }
                int n_scan = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    bool overflow;
                    idx8[k] = 8u * grid_nearest(rec[k], x[2 * k], x[2 * k + 1], (unsigned)K - 1u, overflow, [&](unsigned ci) {
                        const lds_f32x2_t cw = lds_read<lds_f32x2_t>(8u * ci);
                        return make_float2(cw[0], cw[1]);
                    });
                    if (overflow) scan |= 1u << k;
                    n_scan += __popcll(__ballot(active && ((scan >> k) & 1u)));
                }
                decided = n_scan <= bt.dense_above;
                if (decided) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        unsigned long long mask = __ballot(active && ((scan >> k) & 1u));
                        while (mask) {
                            const int src = __ffsll((long long)mask) - 1;
                            mask &= mask - 1;
                            const int bi = wave_exact_scan<cells_least_k(G), cells_codewords(G)>(lane_value(x[2 * k], src), lane_value(x[2 * k + 1], src), 0u, K, ln);
                            if (ln == src) idx8[k] = 8u * (unsigned)bi;
                        }
                    }
                }
            }
#pragma unroll 1
            for (int q = 0; q < 8 / cells_together(G, B) && !decided; ++q) {   // some of the lane's pairs at a time, the rest moved up
                constexpr int P = cells_together(G, B);
                float x0[P], x1[P];
                unsigned got[P];
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    x0[p] = x[2 * p];
                    x1[p] = x[2 * p + 1];
                }
                nearest_of_all<P, (G == 64 ? 1 : 2), cells_least_k(G), cells_codewords(G)>(x0, x1, got, active ? (1u << P) - 1u : 0u, 0u, K, ln);
#pragma unroll
                for (int e = 0; e < 16 - 2 * P; ++e) x[e] = x[e + 2 * P];
#pragma unroll
                for (int k = 0; k < 8 - P; ++k) idx8[k] = idx8[k + P];
#pragma unroll
                for (int p = 0; p < P; ++p) idx8[8 - P + p] = got[p];
            }
            if (active) store_fields<3>(M.packed + (int64_t)row * M.row_bytes, M.row_bytes, M.d_in, c, idx8, bits);
        }
    }
}

// More than the default 64 KB of LDS per workgroup has to be asked for: a host-side setting per kernel and device, made
// once per kernel instantiation and device (the devices' bits of `done`).
template <int DTYPE, int B, int G, bool OWN> static bool cells_allow_large_lds(int dev) {
    static std::atomic<uint64_t> done{0};
    if (dev < 0 || dev >= 64) return false;
    if (done.load(std::memory_order_acquire) & (1ull << dev)) return true;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_encode_cells<DTYPE, B, G, true, OWN>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)cells_lds_bytes(G, OWN));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    done.fetch_or(1ull << dev, std::memory_order_release);
    return true;
}

template <int DTYPE, int B, int G>
static hipError_t launch_cells_dbg(CellsBatch &bt, hipStream_t stream) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1) {
        (void)hipGetLastError();
        return hipErrorNotSupported;
    }
    int64_t items = 0, rows = 0;
    int norm_blocks = 0, most_slabs = 1;
    int64_t own_bytes = 0;
    for (int i = 0; i < bt.n; ++i) {
        CellsMat &M = bt.m[i];
        rows += M.d_out;
        items += (int64_t)M.d_out * M.n_slabs;
        M.log_slabs = __builtin_ctz((unsigned)M.n_slabs);
        M.own_norms = M.slab_sums && cells_shares_rows(DTYPE, M.n_slabs, M.d_in);
        if (M.own_norms) own_bytes += (int64_t)M.d_out * M.d_in * (DTYPE == 0 ? 4 : 2) / cells_own_parts(M.log_slabs);
    }
    const bool direct_launch = G == 128 && items <= CELLS_DIRECT_MAX_ITEMS, own = !direct_launch && own_bytes >= CELLS_OWN_MIN_BYTES;
    for (int i = 0; i < bt.n && !own; ++i) bt.m[i].own_norms = 0;
    const int per_wave = rows >= CELLS_ROWS_TOGETHER ? 4 : 1;
    for (int i = 0; i < bt.n; ++i) {
        const CellsMat &M = bt.m[i];
        bt.norm_begin[i] = norm_blocks;
        if (!M.own_norms) norm_blocks += (M.d_out + CP_WAVES * per_wave - 1) / (CP_WAVES * per_wave);
        if (M.n_slabs > most_slabs) most_slabs = M.n_slabs;
    }
    for (int i = bt.n; i <= QAMW_ENCODE_MAX_BATCH; ++i) bt.norm_begin[i] = norm_blocks;
    const unsigned prep = (unsigned)((G / 8) * (G / 8) + norm_blocks);
    auto prepare = [&]() {
        if (per_wave == 4) hipLaunchKernelGGL((k_cells_prepare<DTYPE, G, 4>), dim3(prep), dim3(CP_THREADS), 0, stream, bt);
        else hipLaunchKernelGGL((k_cells_prepare<DTYPE, G, 1>), dim3(prep), dim3(CP_THREADS), 0, stream, bt);
        return hipGetLastError();
    };
    if constexpr (G == 128) {
        if (direct_launch) {
            constexpr int DIRECT_WAVES = CELLS_DIRECT_THREADS / WAVE;
            const unsigned direct = (unsigned)((items + most_slabs + DIRECT_WAVES - 1) / DIRECT_WAVES);   // an item per wave, whole rows
            const hipError_t e = prepare();
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((k_encode_cells<DTYPE, B, G, false, false>), dim3(direct), dim3(CELLS_DIRECT_THREADS),
                               (size_t)cells_codewords(G) * sizeof(float2), stream, bt);
            return hipGetLastError();
        }
    }
    auto search = [&](auto own_norms) {
        constexpr bool OWN = decltype(own_norms)::value;
        constexpr int WAVES = cells_threads(G, OWN) / WAVE;
        constexpr size_t lds = cells_lds_bytes(G, OWN);
        if (lds > 64 * 1024 && !cells_allow_large_lds<DTYPE, B, G, OWN>(dev)) return hipErrorNotSupported;
        const int64_t blocks = std::min((items + WAVES - 1) / WAVES, (int64_t)cus * cells_per_cu(G, OWN, DTYPE));
        if (blocks * WAVES < most_slabs) return hipErrorNotSupported;   // every wave keeps to one slab: at least a row's worth of waves
        const hipError_t e = prepare();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_encode_cells<DTYPE, B, G, true, OWN>), dim3((unsigned)blocks), dim3(cells_threads(G, OWN)), lds, stream, bt);
        return hipGetLastError();
    };
    return own ? search(std::true_type{}) : search(std::false_type{});
}

template <int DTYPE, int B>
static hipError_t launch_cells_db(CellsBatch &bt, hipStream_t stream) {
    switch (cells_side(bt.bits)) {
        case 128: return launch_cells_dbg<DTYPE, B, 128>(bt, stream);
        case 96: return launch_cells_dbg<DTYPE, B, 96>(bt, stream);
        default: return launch_cells_dbg<DTYPE, B, 64>(bt, stream);
    }
}

template <int DTYPE>
static hipError_t launch_cells_d(CellsBatch &bt, int block, hipStream_t stream) {
    switch (block) {
        case 64: return launch_cells_db<DTYPE, 64>(bt, stream);
        case 128: return launch_cells_db<DTYPE, 128>(bt, stream);
        case 256: return launch_cells_db<DTYPE, 256>(bt, stream);
        case 512: return launch_cells_db<DTYPE, 512>(bt, stream);
        case 1024: return launch_cells_db<DTYPE, 1024>(bt, stream);
        default: return hipErrorNotSupported;
    }
}

size_t encode_cells_bytes(int bits) { return bits <= 11 ? (size_t)cells_side(bits) * cells_side(bits) * sizeof(uint2) : 0; }

// n <= QAMW_ENCODE_MAX_BATCH matrices that share codebook, bits, block and element type; table: encode_cells_bytes(bits)
// bytes of device scratch, 16-byte aligned.  Returns hipErrorNotSupported (nothing launched) when any item is outside the
// kernel's range.
hipError_t launch_encode_cells(const EncodeItem *items, int n, int dtype, const Problem &p, void *table, const SearchGridView *grid) {
    if (n < 1 || n > QAMW_ENCODE_MAX_BATCH || p.bits > 11 || !table || (reinterpret_cast<uintptr_t>(table) & 15) ||
        (reinterpret_cast<uintptr_t>(p.codebook) & 7))
        return hipErrorNotSupported;
    const int unit = p.block > 16 ? p.block : 16;
    CellsBatch bt;
    int64_t items_total = 0;
    for (int i = 0; i < n; ++i) {
        Problem q = p;
        q.chan_scale = items[i].chan_scale;
        q.signs = items[i].signs;
        q.pair_sigma = items[i].pair_sigma;
        if (p.block < 64 || items[i].d_in % unit || !front_alignment_ok(items[i].W, dtype, items[i].ldw, q)) return hipErrorNotSupported;
        CellsMat &M = bt.m[i];
        M.W = items[i].W;
        M.ldw = items[i].ldw;
        M.chan_scale = items[i].chan_scale;
        M.signs = items[i].signs;
        M.pair_sigma = items[i].pair_sigma;
        M.norms = items[i].norms;
        M.packed = items[i].packed;
        M.row_bytes = (((int64_t)(items[i].d_in / 2) * p.bits + 31) / 32) * 4;
        M.d_in = items[i].d_in;
        M.d_out = items[i].d_out;
        M.n_slabs = (items[i].d_in + 1023) / 1024;
        M.g_default = (float)std::sqrt((double)items[i].d_in);
        // The norms of the call without scratch, to the bit: in the order of the kernel that serves it (the pruned search's, the
        // general kernels' and those of longer rows come from a launch of their own).
        q.d_in = items[i].d_in;
        M.slab_sums = !grid && fused_norms_supported(q) && (mfma_encode_supported(q) || fast_encode_supported(q)) &&
                      (reinterpret_cast<uintptr_t>(p.codebook) & 15) == 0;
        if ((int64_t)M.d_out * M.n_slabs > 0x3fffffff) return hipErrorNotSupported;
        items_total += (int64_t)M.d_out * M.n_slabs;
    }
    // Two launches of 11 us at the least: codebooks of up to 32 points are searched whole sooner in small matrices (32 points,
    // bf16, us whole / table: 1024 x 2048, 2048 items, 12.9 / 14.9; 2048 x 2048 20.8 / 15.4).  With 64 points and more the table
    // wins from the smallest matrix on (48 x 512: 17.3 / 14.0; 2048 points 83 / 17).  The pruned search's caller has a table in
    // hand, good for a little more (2048 points, us caller's / this one: 256 x 2048, 512 items, 16.6 / 18.7; 512 x 2048 21.9 / 17.8).
    if (grid ? items_total < CELLS_GRID_MIN_ITEMS : p.bits < 6 && items_total < CELLS_MIN_ITEMS) return hipErrorNotSupported;
    for (int i = n; i < QAMW_ENCODE_MAX_BATCH; ++i) bt.m[i] = bt.m[0];
    bt.n = n;
    bt.bits = p.bits;
    bt.K = p.K;
    bt.inv_sqrt_block = p.inv_sqrt_block;
    bt.half_per_sum = cells_half_per_sum(p.bits);
    bt.dense_above = cells_dense_above(p.K, dtype == 1);
    bt.grid = nullptr;
    bt.grid_side = 0;
    if (grid && p.K > 32) {                                     // (up to 32 codewords all distances are as soon computed)
        bt.grid = static_cast<const uint32_t *>(grid->table);
        bt.grid_side = grid->G;
    }
    bt.codebook = p.codebook;
    bt.table = static_cast<uint2 *>(table);
    return dtype == 0 ? launch_cells_d<0>(bt, p.block, p.stream) : launch_cells_d<1>(bt, p.block, p.stream);
}

}  // namespace qamw
