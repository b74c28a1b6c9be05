// The cell table of the pruned nearest-codeword search (Sec. 3.1 / Sec. 3.5), made on the device: shared by the encoder
// and the device's codebook training.
//
// A square [-R, R]^2 is cut into G x G cells; a cell's record lists, in ascending index order, every codeword that can be
// nearest to a point of the cell, at most five, or says that the whole codebook has to be searched.
//
// The cells are narrow in the middle, where a codebook of Gaussian pairs is dense, and wide at the edge: with s = x / 2R + 1/2,
// kept between 0 and 1, a pair's cell is the integer nearest to (G - 1) s^2 (3 - 2s) in each coordinate, two more multiply-adds
// than cells of one width.  In the middle that is as fine as 1.5 G cells of one width: for 2^11 points and G = 128 2.5 candidates
// on average over the pairs, five for 0.14 % of them, more for 0.001 % (one width and R = 4: 3.1, 3.9 % and 0.05 %).  So four
// candidates are read out of every record, and the fifth only where a wave holds one.
//
// The outermost cells reach to CELLS_FAR times R, and not only to R: strips that cross few codewords' neighbourhoods.  Pairs beyond
// that, and the four corners, are searched for in the whole codebook.
//
// R is 17/16 of `half`, which follows the codebook's scale: 4 where the codewords lie as those of a Lloyd codebook of the unit
// Gaussian, in proportion to their mean |coordinate| otherwise, rounded to four significant bits.  Every workgroup that makes a
// part of the table finds the same, the first leaves it in the table (cells_put_half).  A fixed square is of no use to a codebook
// of another scale: 4096 x 4096 bf16, 2048 points, codebook and pairs / 16: 3960 us with [-4, 4)^2, where the search over the whole
// codebook takes 615; 36 so.
//
// Which codewords a cell lists.  For two codewords a and c the difference |x - c|^2 - |x - a|^2 is linear in x, so on a
// box of half-widths w, v around m it is at least |m - c|^2 - |m - a|^2 - 2 (w |c.x - a.x| + v |c.y - a.y|).  c is left out
// when that exceeds a margin: then a is nearer at every point of the box, also after the roundings of the fp32 distances
// (relative error below 2.4e-7 each; the margin is 4e-6 of the two squared distances and 1e-5 (w^2 + v^2)).  As `a` serve the
// codewords nearest and second nearest to m: for a Lloyd codebook of the Gaussian that leaves the same lists as testing
// all pairs.  The lists are found top down -- 8 x 8 cells, 4 x 4 cells, single cells -- and each level searches only its parent's
// list.
#pragma once
#include "qamw_front.hpp"

namespace qamw {

constexpr int CELLS_LIST = 5;                                  // candidates of a record
// A record's two words: the first four candidates' byte offsets in the codebook, index times 8, in the bits 3 to 13 of the four
// 16-bit halves, where one instruction takes them out; the fifth's index in what is left, see cells_fifth(); and
constexpr uint32_t CELLS_FIFTH = 0x80000000u;                  // in the upper word: five candidates;
constexpr uint32_t CELLS_SCAN = 0x40000000u;                   //   decided by the whole codebook;
constexpr uint32_t CELLS_BORDER = 0x00004000u;                 //   a cell of the edge: of pairs within CELLS_FAR
constexpr uint32_t CELLS_OFFSET = 0x3ff8u;
constexpr float CELLS_REACH = 1.0625f, CELLS_FAR = 1.25f;      // R over half; how far the outermost cells reach, over R

// Cells per side.  Four cells per codeword spacing at the centre of a Lloyd codebook keep the lists within a record;
// the LDS holds 128 x 128 records beside 2048 codewords.
constexpr int cells_side(int bits) { return bits >= 11 ? 128 : bits == 10 ? 96 : 64; }

// half over the sum of the magnitudes of n = min(K, CP_SAMPLE) codewords' coordinates, so that a Lloyd codebook of the unit
// Gaussian with K = 2^bits points gets 4 after the rounding, from 3.875 to 4.25: 4 over 2 n times 1 / 1.015 of the mean
// |coordinate| of such a codebook's sample (qamw_train_codebook with 2^14 to 2^20 samples and 10 to 200 iterations: raw values
// of 4.01 to 4.18 from 7 bits on).
constexpr int CP_SAMPLE = 256;                                 // 32 evenly spread runs of eight: a cache line each
inline float cells_half_per_sum(int bits) {
    constexpr float mean[11] = {0.52f, 0.708f, 0.81f, 0.89f, 0.97f, 1.016f, 1.058f, 1.085f, 1.076f, 1.078f, 1.071f};
    const int n = 1 << bits < CP_SAMPLE ? 1 << bits : CP_SAMPLE;
    return 4.0f / (mean[bits - 1] * 2.0f * (float)n);
}
// half is kept in the first record, a corner's, which has no candidates: its upper 12 bits from bit 3 on.
__device__ __forceinline__ uint32_t cells_put_half(float half) { return (__float_as_uint(half) >> 20) << 3; }
__device__ __forceinline__ float cells_half(const uint2 *table) { return __uint_as_float((table[0].x >> 3) << 20); }
// 1 / 2R, one rounding or two off (the boxes' slack is 2^-16 of half), in a scalar register.
__device__ __forceinline__ float wave_uniform(float v) {
    asm volatile("" : "+v"(v));                                 // (left in a vector register where the compiler knows that it is uniform)
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}
__device__ __forceinline__ float cells_inv_span(float half) { return wave_uniform((0.5f / CELLS_REACH) * __builtin_amdgcn_rcpf(wave_uniform(half))); }
// Up to where a record of the edge holds.
__device__ __forceinline__ float cells_far(float half) { return wave_uniform(CELLS_REACH * CELLS_FAR * half); }

// The cells' edges over half: of cell i from at[i] to at[i + 1].
template <int G> struct CellsEdges {
    float at[G + 1];
    constexpr CellsEdges() : at() {
        for (int i = 1; i < G; ++i) {
            const double t = (i - 0.5) / (G - 1);
            double lo = 0.0, hi = 1.0;                          // s^2 (3 - 2s) = t
            for (int k = 0; k < 50; ++k) {
                const double s = 0.5 * (lo + hi);
                (s * s * (3.0 - 2.0 * s) < t ? lo : hi) = s;
            }
            at[i] = (float)((lo + hi - 1.0) * (double)CELLS_REACH);
        }
        at[0] = -CELLS_REACH * CELLS_FAR;
        at[G] = CELLS_REACH * CELLS_FAR;
    }
};
template <int G> static __constant__ const CellsEdges<G> cells_edges{};

// ------------------------------------------------------------------------------------------------ the table
constexpr int CP_THREADS = 256;
constexpr int CP_WAVES = CP_THREADS / WAVE;
constexpr int CP_REGION_LIST = 512;                            // candidates of 8 x 8 cells (150 at most for 2^11 Lloyd points)
constexpr int CP_BLOCK_LIST = 128;                             // candidates of 4 x 4 cells (70)
constexpr int CP_PER_THREAD = 2048 / CP_THREADS;

struct CellsBox {
    float mx, my, wx, wy;                                       // centre and half-widths
};
// n x n cells from (ix, iy) on
template <int G> __device__ __forceinline__ CellsBox cells_box(int ix, int iy, int n, float half) {
    const float slack = half * 0x1p-16f;                        // the fp32 roundings of the edges and of the cell lookup (2e-6)
    const float x0 = cells_edges<G>.at[ix] * half, x1 = cells_edges<G>.at[ix + n] * half;
    const float y0 = cells_edges<G>.at[iy] * half, y1 = cells_edges<G>.at[iy + n] * half;
    return {0.5f * (x0 + x1), 0.5f * (y0 + y1), 0.5f * (x1 - x0) + slack, 0.5f * (y1 - y0) + slack};
}
// Is codeword c farther than codeword a at every point of the box?  dc2, da2: their squared distances from its centre.
__device__ __forceinline__ bool cells_dominated(float2 c, float dc2, float2 a, float da2, const CellsBox &b) {
    const float reach = 2.00002f * (b.wx * fabsf(c.x - a.x) + b.wy * fabsf(c.y - a.y));
    return dc2 - da2 > reach + 4e-6f * (dc2 + da2) + 1e-5f * (b.wx * b.wx + b.wy * b.wy);
}
__device__ __forceinline__ float cells_dist2(const CellsBox &b, float2 c) {
    const float ex = b.mx - c.x, ey = b.my - c.y;
    return ex * ex + ey * ey;
}

// The lanes' smallest distance and its codeword, in every lane.
__device__ __forceinline__ void wave_nearest(float &d, float2 &c) {
    const float least = wave_min(d);
    const int at = __ffsll((long long)__ballot(d == least)) - 1;
    d = least;
    c = make_float2(lane_value(c.x, at), lane_value(c.y, at));
}

// What a thread of a workgroup that makes a part of the table holds: a run of consecutive codewords, and its lane's part of
// the sample that R is found from (the same in every wave of every workgroup).
struct CellsPoints {
    float2 run[CP_PER_THREAD], sample[CP_SAMPLE / WAVE];
};
// point(i): the i-th of K codewords
template <class Point> __device__ __forceinline__ CellsPoints cells_points(int K, Point point) {
    CellsPoints p;
    const int lane = threadIdx.x & (WAVE - 1), per = (K + CP_THREADS - 1) / CP_THREADS, first = (int)threadIdx.x * per;
    const int spread = max(K / CP_SAMPLE, 1);
#pragma unroll
    for (int q = 0; q < CP_SAMPLE / WAVE; ++q) p.sample[q] = point(min(((lane >> 3) + 8 * q) * 8 * spread + (lane & 7), K - 1));
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) p.run[j] = point(j < per && first + j < K ? first + j : 0);
    return p;
}

// Candidate lists of 8 x 8 cells by one workgroup; wave w takes their w-th quarter of 4 x 4 cells.
//   Bound by latency, one workgroup per CU: hence minima and prefix sums by DPP moves and ballots instead of shuffles, and
// LDS reads four to sixteen at a time (2048 points, 16 x 16 regions: 7.8 us; with a cell's candidates read four at a time, twice,
// and their indices one by one 9.1; 14 x 14 with shuffles and one read at a time 11.3).
template <int G>
__device__ __forceinline__ void cells_build_region(const CellsPoints &points, int K, float half_per_sum, uint2 *table, int region) {
    __shared__ float2 reg_c[CP_REGION_LIST];
    __shared__ uint16_t reg_i[CP_REGION_LIST];
    __shared__ float2 blk_c[CP_WAVES][CP_BLOCK_LIST];
    __shared__ uint16_t blk_i[CP_WAVES][CP_BLOCK_LIST];
    __shared__ uint16_t rec_i[CP_WAVES][16][8];
    __shared__ float red_d[CP_WAVES];
    __shared__ float2 red_c[CP_WAVES];
    __shared__ int red_n[CP_WAVES];
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x >> 6;
    const int x0 = (region % (G / 8)) * 8, y0 = (region / (G / 8)) * 8;

    // ---- 8 x 8 cells: every thread holds a run of consecutive codewords
    const int per = (K + CP_THREADS - 1) / CP_THREADS, first = (int)threadIdx.x * per;
    const float2 (&c)[CP_PER_THREAD] = points.run;
    float d2[CP_PER_THREAD];
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < CP_SAMPLE / WAVE; ++q) s += q * WAVE + lane < K ? fabsf(points.sample[q].x) + fabsf(points.sample[q].y) : 0.0f;
    s = wave_add(s) * half_per_sum;
    // squares of distances inside a cell stay normal numbers
    const float half = __uint_as_float((__float_as_uint(fminf(fmaxf(s, 0x1p-40f), 0x1p40f)) + 0x80000u) & 0xFFF00000u);
    CellsBox box = cells_box<G>(x0, y0, 8, half);
    float nd = 3.0e38f;
    float2 nc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) {
        d2[j] = cells_dist2(box, c[j]);
        if (d2[j] < nd) {
            nd = d2[j];
            nc = c[j];
        }
    }
    wave_nearest(nd, nc);
    if (lane == 0) {
        red_d[wid] = nd;
        red_c[wid] = nc;
    }
    __syncthreads();
    nd = red_d[0];
    nc = red_c[0];
#pragma unroll
    for (int q = 1; q < CP_WAVES; ++q) {
        if (red_d[q] < nd) {
            nd = red_d[q];
            nc = red_c[q];
        }
    }
    unsigned keep = 0;
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j)
        if (j < per && first + j < K && !cells_dominated(c[j], d2[j], nc, nd, box)) keep |= 1u << j;
    int below = __popc(keep);                                   // inclusive sum over the lanes up to this one
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) {
        const unsigned long long mask = __ballot((keep >> j) & 1u);
        below += __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
    }
    if (lane == WAVE - 1) red_n[wid] = below;
    __syncthreads();
    int at = below - __popc(keep), n_reg = 0;
#pragma unroll
    for (int q = 0; q < CP_WAVES; ++q) {
        if (q < wid) at += red_n[q];
        n_reg += red_n[q];
    }
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) {
        if ((keep >> j) & 1u) {
            if (at < CP_REGION_LIST) {
                reg_c[at] = c[j];
                reg_i[at] = (uint16_t)(first + j);
            }
            ++at;
        }
    }
    __syncthreads();
    bool too_long = n_reg > CP_REGION_LIST;
    if (too_long) n_reg = 0;

    // ---- 4 x 4 cells: the wave's lanes share the region's candidates
    const int bx = x0 + 4 * (wid & 1), by = y0 + 4 * (wid >> 1);
    box = cells_box<G>(bx, by, 4, half);
    nd = 3.0e38f;
    constexpr int RUNS = CP_REGION_LIST / WAVE;
    float2 ce[RUNS];
    float de[RUNS];
#pragma unroll
    for (int u = 0; u < RUNS; ++u) ce[u] = reg_c[u * WAVE + lane < n_reg ? u * WAVE + lane : 0];
#pragma unroll
    for (int u = 0; u < RUNS; ++u) {
        de[u] = cells_dist2(box, ce[u]);
        if (u * WAVE + lane < n_reg && de[u] < nd) {
            nd = de[u];
            nc = ce[u];
        }
    }
    wave_nearest(nd, nc);
    int n_blk = 0;
#pragma unroll
    for (int u = 0; u < RUNS; ++u) {
        if (u * WAVE >= n_reg) break;
        const bool k = u * WAVE + lane < n_reg && !cells_dominated(ce[u], de[u], nc, nd, box);
        const unsigned long long mask = __ballot(k);
        const int pos = n_blk + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
        if (k && pos < CP_BLOCK_LIST) {
            blk_c[wid][pos] = ce[u];
            blk_i[wid][pos] = reg_i[u * WAVE + lane];
        }
        n_blk += __popcll(mask);
    }
    too_long = too_long || n_blk > CP_BLOCK_LIST;
    if (too_long) n_blk = 0;
    __syncthreads();

    // ---- single cells: four lanes per cell, each a quarter of the block's candidates
    const int cell = lane >> 2, part = lane & 3;
    const int ix = bx + (cell & 3), iy = by + (cell >> 2);
    box = cells_box<G>(ix, iy, 1, half);
    const int quarter = (n_blk + 3) >> 2, e_begin = part * quarter, e_end = min(n_blk, e_begin + quarter);
    // The quarter's candidates in registers, in one round of LDS reads; those of a longer list are read again in both passes.
    constexpr int HELD = CP_BLOCK_LIST / 8;
    float2 held[HELD];
    float dh[HELD];
#pragma unroll
    for (int q = 0; q < HELD; ++q) held[q] = blk_c[wid][min(e_begin + q, CP_BLOCK_LIST - 1)];
    float da = 3.0e38f, db = 3.0e38f;                           // nearest and second nearest
    float2 ca = make_float2(0.0f, 0.0f), cb = ca;
    auto rank = [&](float2 c, float d) {
        const bool first_of_all = d < da, second = d < db;
        cb.x = first_of_all ? ca.x : second ? c.x : cb.x;
        cb.y = first_of_all ? ca.y : second ? c.y : cb.y;
        db = first_of_all ? da : second ? d : db;
        ca.x = first_of_all ? c.x : ca.x;
        ca.y = first_of_all ? c.y : ca.y;
        da = first_of_all ? d : da;
    };
#pragma unroll
    for (int q = 0; q < HELD; ++q) {
        dh[q] = e_begin + q < e_end ? cells_dist2(box, held[q]) : 3.0e38f;
        rank(held[q], dh[q]);
    }
    for (int e = e_begin + HELD; e < e_end; ++e) rank(blk_c[wid][e], cells_dist2(box, blk_c[wid][e]));
    auto merge = [&](float oda, float odb, float2 oca, float2 ocb) {
        // each side's two, sorted: the first is the smaller head, the second the smaller of the other head and its own second
        const bool swap = oda < da;
        const float hd = swap ? da : oda, td = swap ? odb : db;
        const float2 hc = swap ? ca : oca, tc = swap ? ocb : cb;
        if (swap) {
            da = oda;
            ca = oca;
        }
        const bool head = hd < td;
        db = head ? hd : td;
        cb = head ? hc : tc;
    };
    merge(dpp_move<DPP_XOR1>(da), dpp_move<DPP_XOR1>(db), make_float2(dpp_move<DPP_XOR1>(ca.x), dpp_move<DPP_XOR1>(ca.y)),
          make_float2(dpp_move<DPP_XOR1>(cb.x), dpp_move<DPP_XOR1>(cb.y)));
    merge(dpp_move<DPP_XOR2>(da), dpp_move<DPP_XOR2>(db), make_float2(dpp_move<DPP_XOR2>(ca.x), dpp_move<DPP_XOR2>(ca.y)),
          make_float2(dpp_move<DPP_XOR2>(cb.x), dpp_move<DPP_XOR2>(cb.y)));
    unsigned kept = 0;                                          // bit e - e_begin (a quarter is at most 32 candidates)
    auto keeps = [&](float2 c, float d) {
        return !(cells_dominated(c, d, ca, da, box) || (db < 3.0e38f && cells_dominated(c, d, cb, db, box)));
    };
#pragma unroll
    for (int q = 0; q < HELD; ++q)
        if (e_begin + q < e_end && keeps(held[q], dh[q])) kept |= 1u << q;
    for (int e = e_begin + HELD; e < e_end; ++e)
        if (keeps(blk_c[wid][e], cells_dist2(box, blk_c[wid][e]))) kept |= 1u << (e - e_begin);
    const int mine = __popc(kept);
    const int n0 = dpp_move<dpp_quad_lane(0)>(mine), n1 = dpp_move<dpp_quad_lane(1)>(mine), n2 = dpp_move<dpp_quad_lane(2)>(mine);
    int before = (part > 0 ? n0 : 0) + (part > 1 ? n1 : 0) + (part > 2 ? n2 : 0);
    const int total = n0 + n1 + n2 + dpp_move<dpp_quad_lane(3)>(mine);
    while (kept) {
        const int e = e_begin + __ffs((int)kept) - 1;
        kept &= kept - 1u;
        if (before < CELLS_LIST) rec_i[wid][cell][before] = (uint16_t)e;   // the place in the list: its index is read once all are in
        ++before;
    }
    __syncthreads();
    if (part == 0) {
        uint2 r = make_uint2(0u, CELLS_SCAN);
        const bool edge_x = ix == 0 || ix == G - 1, edge_y = iy == 0 || iy == G - 1;
        if (!(edge_x && edge_y) && total >= 1 && total <= CELLS_LIST) {
            unsigned i5[CELLS_LIST];                            // ascending, padded with the first
#pragma unroll
            for (int q = 0; q < CELLS_LIST; ++q) i5[q] = blk_i[wid][rec_i[wid][cell][q < total ? q : 0]];
            r.x = (i5[0] << 3) | (i5[1] << 19) | ((i5[4] & 31u) << 14);
            r.y = (i5[2] << 3) | (i5[3] << 19) | (((i5[4] >> 5) & 15u) << 15) | (i5[4] >> 9) | (total > 4 ? CELLS_FIFTH : 0u) |
                  (edge_x || edge_y ? CELLS_BORDER : 0u);
        }
        if (ix == 0 && iy == 0) r.x = cells_put_half(half);
        table[iy * G + ix] = r;
    }
}


// ------------------------------------------------------------------------------------------------ the search
// Byte offset from table_at of the record of the cell that holds (x0, x1); inv_span: 1 / 2R.
constexpr uint32_t CELLS_MAGIC_BITS = 0x4B000000u;             // 2^23: adding it rounds to an integer, left in the low bits
template <int G> __device__ __forceinline__ uint32_t cells_record_at(float x0, float x1, float inv_span, uint32_t table_at) {
    constexpr float magic = 8388608.0f;
    auto place = [=](float x) {                                 // (G - 1) s^2 (3 - 2s); a NaN is 0
        const float s = fminf(fmaxf(__builtin_fmaf(x, inv_span, 0.5f), 0.0f), 1.0f);
        return __float_as_uint(__builtin_fmaf(s * s, __builtin_fmaf(s, -2.0f * (G - 1), 3.0f * (G - 1)), magic));
    };
    const uint32_t ix = place(x0), iy = place(x1);
    // (iy G + ix) 8 + table_at mod 2^32, the two numbers' exponent bits taken out with the one constant.  Two instructions; three
    // where the compiler multiplies out.
    uint32_t cell;
    if constexpr (G == 128) asm("v_lshl_add_u32 %0, %1, 7, %2" : "=v"(cell) : "v"(iy), "v"(ix));
    else if constexpr (G == 64) asm("v_lshl_add_u32 %0, %1, 6, %2" : "=v"(cell) : "v"(iy), "v"(ix));
    else cell = iy * G + ix;
    return (cell << 3) + (table_at - ((CELLS_MAGIC_BITS * G + CELLS_MAGIC_BITS) << 3));
}
// A candidate as one number: its squared distance's bits above its byte offset in the codebook.  As fp64 values (of finite
// distances, infinity and NaN too) these are in the order of the distance and, of equal ones, of the index, so that the nearest is
// the minimum, one instruction for a comparison and two selections.
__device__ __forceinline__ double cells_candidate(float d, unsigned o) { return __hiloint2double(__float_as_int(d), (int)o); }
__device__ __forceinline__ double cells_nearer(double a, double b) {
    double m;
    asm("v_min_f64 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));     // (as a function of the library it comes with two more that quiet a NaN)
    return m;
}
__device__ __forceinline__ unsigned cells_offset(double candidate) { return (unsigned)__double2loint(candidate); }
__device__ __forceinline__ float cells_distance(double candidate) { return __int_as_float(__double2hiint(candidate)); }

// The record's first four candidates, requested from the codebook in LDS at byte address cb_at, ...
struct CellsFour {
    unsigned o[4];
    lds_f32x2_t c[4];
};
__device__ __forceinline__ void cells_request(CellsFour &f, uint2 rec, uint32_t cb_at) {
    f.o[0] = rec.x & CELLS_OFFSET;
    f.o[1] = (rec.x >> 16) & CELLS_OFFSET;
    f.o[2] = rec.y & CELLS_OFFSET;
    f.o[3] = (rec.y >> 16) & CELLS_OFFSET;
#pragma unroll
    for (int j = 0; j < 4; ++j) f.c[j] = lds_read<lds_f32x2_t>(cb_at + f.o[j]);
}
// ... and the nearest of them.
__device__ __forceinline__ double cells_nearest(const CellsFour &f, float x0, float x1) {
    double d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = cells_candidate(exact_dist2(x0, x1, make_float2(f.c[j][0], f.c[j][1])), f.o[j]);
    return cells_nearer(cells_nearer(d[0], d[1]), cells_nearer(d[2], d[3]));
}
// `best` or the fifth candidate of a record that has one.
__device__ __forceinline__ double cells_fifth(uint2 rec, float x0, float x1, uint32_t cb_at, double best) {
    const unsigned o4 = (((rec.x >> 14) & 31u) | (((rec.y >> 15) & 15u) << 5) | ((rec.y & 3u) << 9)) << 3;
    const lds_f32x2_t c = lds_read<lds_f32x2_t>(cb_at + o4);
    const double nearer = cells_nearer(best, cells_candidate(exact_dist2(x0, x1, make_float2(c[0], c[1])), o4));
    return rec.y & CELLS_FIFTH ? nearer : best;
}
// Whether the whole codebook decides the pair; far: cells_far().  NANS: one coordinate may be a NaN and the other not (the larger of the
// two is the number then).
template <bool NANS> __device__ __forceinline__ bool cells_undecided(uint2 rec, float x0, float x1, float far) {
    const bool near = NANS ? fabsf(x0) <= far && fabsf(x1) <= far : fmaxf(fabsf(x0), fabsf(x1)) <= far;
    return (rec.y & CELLS_SCAN) || ((rec.y & CELLS_BORDER) && !near);
}

// ------------------------------------------------------------------------------------------------ without the table
typedef float cells_f32x16_t __attribute__((ext_vector_type(16)));
typedef __bf16 cells_bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t cells_u32x4_t __attribute__((ext_vector_type(4)));

// (lower half of the wave: a there, upper half: b of the lane 32 below) and (a of the lane 32 above, b)
__device__ __forceinline__ void half_swap(float a, float b, float &lo, float &hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    lo = __uint_as_float(r[0]);
    hi = __uint_as_float(r[1]);
}
// the value of the lane whose number differs in bit 5
__device__ __forceinline__ float other_half(float v, int hs) {
    float lo, hi;
    half_swap(v, v, lo, hi);
    return hs ? lo : hi;
}
__device__ __forceinline__ int other_half(int v, int hs) { return __float_as_int(other_half(__int_as_float(v), hs)); }

// Nearest codewords of P points per lane among all K (a power of two; the codebook in LDS at byte address cb_at): idx[p] = 8
// times the index of the nearest to (x0[p], x1[p]) by exact fp32 squared distance, lowest index on ties.  All lanes call it;
// a point with its bit of `wanted` clear gets some index below K.
//   K >= 64.  A shortlist by matrix instructions, with the operands of the whole-codebook
// encoder (qamw_encode_mfma.hip: scores |c|^2 - 2 x.c from exact bf16 pieces, error at most 2^-19 (|c| + n1)^2, n1 = |x0| +
// |x1|), built from registers: point block 2 p + b are the points p of the lanes of half b.  A chunk is the 16 rows of each of
// CH 32-codeword blocks that a lane holds (two halve the bookkeeping of the loop, one halves the exact distances after it).  bd, the smallest exact distance in the best chunk, bounds the score of whatever is
// nearest: it is not in another chunk if the least score there exceeds bd - |x|^2 by more than the score's error for a
// codeword within sqrt(bd) of x and the roundings.  Else the whole codebook is scanned.  The margin has no scale of its own;
// outside 1e-30 .. 1e30 the products of the pieces are
// no longer exact or overflow, so those points are scanned.
//   For pairs that no table helps.  The whole call, 4096 x 4096 bf16, pairs three times as wide as the codebook: 2048 points,
// one scan after the other 1440 us, so 678 (the encoder without a table 574); 128 points 692 us, so 120 (102).
template <int P, int CH, int K_FROM, int K_TO>
__device__ __forceinline__ void nearest_of_all(const float (&x0)[P], const float (&x1)[P], unsigned (&idx)[P], unsigned wanted, uint32_t cb_at,
                                               int K, int lane) {
    constexpr float BIG = 3.0e38f;
    auto dist = [&](float a, float b, int ci) {
        const lds_f32x2_t c = lds_read<lds_f32x2_t>(cb_at + 8u * (uint32_t)ci);
        return exact_dist2(a, b, make_float2(c[0], c[1]));
    };
    const int j = lane & 31, hs = lane >> 5;
    cells_bf16x8_t bop[2 * P];
    float m1[2 * P], m2[2 * P];
    int best[2 * P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float v[2];
        half_swap(x0[p], x1[p], v[0], v[1]);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            uint32_t h, m, l;
            split3(-2.0f * v[b], h, m, l);
            const cells_u32x4_t u = {pack2(h, m), pack2(h, l), pack2(m, h), 0x3F803F80u};   // h m h l m h 1 1
            bop[2 * p + b] = __builtin_bit_cast(cells_bf16x8_t, u);
            m1[2 * p + b] = m2[2 * p + b] = BIG;
            best[2 * p + b] = 0;
        }
    }
    cells_f32x16_t zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
#pragma unroll 1
    for (int cb = 0; cb < K; cb += 32 * CH) {
        cells_bf16x8_t aop[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const lds_f32x2_t c = lds_read<lds_f32x2_t>(cb_at + 8u * (uint32_t)(cb + 32 * u + j));
            uint32_t h, m, l, nh, nm, nl;
            split3(hs ? c[1] : c[0], h, m, l);
            split3(__builtin_fmaf(c[1], c[1], c[0] * c[0]), nh, nm, nl);
            const cells_u32x4_t ua = {pack2(h, h), pack2(m, h), pack2(m, l), hs ? pack2(nl, 0u) : pack2(nh, nm)};
            aop[u] = __builtin_bit_cast(cells_bf16x8_t, ua);
        }
#pragma unroll
        for (int q = 0; q < 2 * P; ++q) {
            auto min3 = [](float a, float b, float c3) { return __builtin_fminf(__builtin_fminf(a, b), c3); };
            float part[2 * CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const cells_f32x16_t d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aop[u], bop[q], zero, 0, 0, 0);
                const float t0 = min3(d[0], d[1], d[2]), t1 = min3(d[3], d[4], d[5]), t2 = min3(d[6], d[7], d[8]);
                const float t3 = min3(d[9], d[10], d[11]), t4 = min3(d[12], d[13], d[14]);
                part[2 * u] = min3(t0, t1, t2);
                part[2 * u + 1] = min3(t3, t4, d[15]);
            }
            const float least = CH == 1 ? __builtin_fminf(part[0], part[1]) : __builtin_fminf(min3(part[0], part[1], part[2]), part[2 * CH - 1]);
            best[q] = least < m1[q] ? cb : best[q];
            m2[q] = __builtin_amdgcn_fmed3f(m1[q], m2[q], least);              // m1 <= m2: the second smallest
            m1[q] = __builtin_fminf(m1[q], least);
        }
    }
    unsigned unsafe = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float ax[2], ay[2];
        half_swap(x0[p], x0[p], ax[0], ax[1]);
        half_swap(x1[p], x1[p], ay[0], ay[1]);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int q = 2 * p + b;
            const float o1 = other_half(m1[q], hs), o2 = other_half(m2[q], hs);
            const int ob = other_half(best[q], hs);
            const bool other = o1 < m1[q];
            const float least_elsewhere = fminf(fmaxf(m1[q], o1), fminf(m2[q], o2));
            const int first = (other ? ob : best[q]) + 4 * (other ? hs ^ 1 : hs);   // the chunk's rows: first + 8 q + t
            float bd = BIG;
            int bi = first;
#pragma unroll
            for (int i = 0; i < 8 * CH; ++i) {                  // this lane's half of them, ascending
                const int ci = first + 32 * (i >> 3) + 16 * hs + 8 * ((i >> 2) & 1) + (i & 3);
                const float dd = dist(ax[b], ay[b], ci);
                if (dd < bd) {
                    bd = dd;
                    bi = ci;
                }
            }
            const float od = other_half(bd, hs);
            const int oi = other_half(bi, hs);
            if (od < bd || (od == bd && oi < bi)) {
                bd = od;
                bi = oi;
            }
            const float n1 = fabsf(ax[b]) + fabsf(ay[b]), xx = __builtin_fmaf(ay[b], ay[b], ax[b] * ax[b]);
            const float reach = 2.0f * n1 + sqrtf(bd);
            const float margin = 4e-6f * reach * reach;         // 2^-19 (|c| + n1)^2 with |c| <= n1 + sqrt(bd), and 2e-6 (bd + xx)
            const bool safe = least_elsewhere - (bd - xx) > margin && margin > 1e-30f && margin < 1e30f;
            if (hs == b) {
                idx[p] = 8u * (unsigned)bi;
                if (!safe) unsafe |= 1u << p;
            }
        }
    }
    unsafe &= wanted;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        unsigned long long mask = __ballot((unsafe >> p) & 1u);
        while (mask) {
            const int src = __ffsll((long long)mask) - 1;
            mask &= mask - 1;
            const int bi = wave_exact_scan<K_FROM, K_TO>(lane_value(x0[p], src), lane_value(x1[p], src), cb_at, K, lane);
            if (lane == src) idx[p] = 8u * (unsigned)bi;
        }
    }
}
// Above this many undecided ones of a wave's 512 pairs a search of all of them without the table is sooner done than one scan of the
// codebook after the other.  From pairs 2.2, 2.5, 2.8 and 3.2 times as wide as the codebook (24, 42, 67 and 105 undecided), us with all
// scanned / none, 12288 x 4096 bf16: 6 bits 174 257 369 545 / 290; 8 bits 230 359 542 815 / 438; 9 bits 236 371 558 846 / 640;
// 10 bits 305 475 733 1115 / 1140; 11 bits 488 818 1295 2004 / 2010.  The two meet at 50, 53, 78, 106 and 105; in 4096 x 4096 at 50, 52, 72, 95
// and 92; with fp32 weights at 38 to 41 (6 to 8 bits), 62 (9) and 96 to 105 (11).  From 512 codewords on a scan requests eight a lane at once.
constexpr int cells_dense_above(int K, bool bf16) {
    return K >= 1024 ? 98 : K >= 512 ? (bf16 ? 72 : 62) : K > 32 ? (bf16 ? 50 : 39) : 16;
}

}  // namespace qamw
