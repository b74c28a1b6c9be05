// The cell table of the pruned nearest-codeword search (Sec. 3.1 / Sec. 3.5), made on the device: shared by the encoder
// and the device's codebook training.
//
// The square [-4, 4)^2 is cut into G x G cells; a cell's record lists, in ascending index order, every codeword that can be
// nearest to a point of the cell, at most five, or says that the whole codebook has to be searched.
//
// Which codewords a cell lists.  For two codewords a and c the difference |x - c|^2 - |x - a|^2 is linear in x, so on a
// box of half-width w around m it is at least |m - c|^2 - |m - a|^2 - 2 w (|c.x - a.x| + |c.y - a.y|).  c is left out
// when that exceeds a margin: then a is nearer at every point of the box, also after the roundings of the fp32 distances
// (relative error below 2.4e-7 each; the margin is 4e-6 of the two squared distances and 1e-5 w^2).  As `a` serve the
// codewords nearest and second nearest to m: for a Lloyd codebook of the Gaussian that leaves the same lists as testing
// all pairs (2^11 points, G = 128: 3.1 candidates on average over the pairs, six for 0.05 % of them, never more).  The lists are
// found top down -- 8 x 8 cells, 4 x 4 cells, single cells -- and each level searches only its parent's list.
#pragma once
#include "qamw_front.hpp"

namespace qamw {

constexpr float CELLS_HALF = 4.0f;                             // the table covers [-4, 4)^2 less a border of one cell
constexpr int CELLS_LIST = 5;                                  // candidates of a record
constexpr uint32_t CELLS_SCAN = 0x80000000u;                   // in the record's upper word: decided by the whole codebook
constexpr uint32_t CELLS_MORE = 1u;                            // in its lower word: more than three candidates


// Cells per side.  Four cells per codeword spacing at the centre of a Lloyd codebook keep the lists within a record;
// the LDS holds 128 x 128 records beside 2048 codewords.
constexpr int cells_side(int bits) { return bits >= 11 ? 128 : bits == 10 ? 96 : 64; }

// ------------------------------------------------------------------------------------------------ the table
constexpr int CP_THREADS = 256;
constexpr int CP_WAVES = CP_THREADS / WAVE;
constexpr int CP_REGION_LIST = 512;                            // candidates of 8 x 8 cells (200 at most for 2^11 Lloyd points)
constexpr int CP_BLOCK_LIST = 128;                             // candidates of 4 x 4 cells (55)
constexpr int CP_PER_THREAD = 2048 / CP_THREADS;

// Is codeword c farther than codeword a at every point of the box of half-width w around m?  dc2, da2: their squared
// distances from m.
__device__ __forceinline__ bool cells_dominated(float2 c, float dc2, float2 a, float da2, float w) {
    const float reach = 2.00002f * w * (fabsf(c.x - a.x) + fabsf(c.y - a.y));
    return dc2 - da2 > reach + 4e-6f * (dc2 + da2) + 1e-5f * w * w;
}
__device__ __forceinline__ float cells_dist2(float mx, float my, float2 c) {
    const float ex = mx - c.x, ey = my - c.y;
    return ex * ex + ey * ey;
}

// The lanes' smallest distance and its codeword, in every lane.
__device__ __forceinline__ void wave_nearest(float &d, float2 &c) {
    const float least = wave_min(d);
    const int at = __ffsll((long long)__ballot(d == least)) - 1;
    d = least;
    c = make_float2(lane_value(c.x, at), lane_value(c.y, at));
}

// Candidate lists of 8 x 8 cells by one workgroup; wave w takes their w-th quarter of 4 x 4 cells.
// stopped_at, t: nothing is made once *stopped_at < t (looked at while the codewords are on their way).
//   Bound by latency, one workgroup per CU: hence minima and prefix sums by DPP moves and ballots instead of shuffles, and
// LDS reads four to eight at a time (2048 points, 16 x 16 regions: 8.2 us; 14 x 14 with shuffles and one read at a time 11.3).
template <int G>
__device__ __forceinline__ void cells_build_region(const float *codebook, int K, uint2 *table, int region, const int *stopped_at = nullptr,
                                                   int t = 0) {
    __shared__ float2 reg_c[CP_REGION_LIST];
    __shared__ uint16_t reg_i[CP_REGION_LIST];
    __shared__ float2 blk_c[CP_WAVES][CP_BLOCK_LIST];
    __shared__ uint16_t blk_i[CP_WAVES][CP_BLOCK_LIST];
    __shared__ uint16_t rec_i[CP_WAVES][16][8];
    __shared__ float red_d[CP_WAVES];
    __shared__ float2 red_c[CP_WAVES];
    __shared__ int red_n[CP_WAVES];
    constexpr float h = 2.0f * CELLS_HALF / G;
    constexpr float slack = CELLS_HALF / 524288.0f;            // the fp32 roundings of the centres and of the cell lookup
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x >> 6;
    const float2 *cbk = reinterpret_cast<const float2 *>(codebook);
    const int x0 = (region % (G / 8)) * 8, y0 = (region / (G / 8)) * 8;

    // ---- 8 x 8 cells: every thread holds a run of consecutive codewords
    const int per = (K + CP_THREADS - 1) / CP_THREADS, first = (int)threadIdx.x * per;
    float2 c[CP_PER_THREAD];
    float d2[CP_PER_THREAD];
    const int stop = stopped_at ? *stopped_at : t;
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) c[j] = cbk[j < per && first + j < K ? first + j : 0];
    if (stop < t) return;
    float mx = ((float)x0 + 3.5f - 0.5f * G) * h, my = ((float)y0 + 3.5f - 0.5f * G) * h, w = 4.0f * h + slack;
    float nd = 3.0e38f;
    float2 nc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) {
        d2[j] = cells_dist2(mx, my, c[j]);
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
        if (j < per && first + j < K && !cells_dominated(c[j], d2[j], nc, nd, w)) keep |= 1u << j;
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
    mx = ((float)bx + 1.5f - 0.5f * G) * h;
    my = ((float)by + 1.5f - 0.5f * G) * h;
    w = 2.0f * h + slack;
    nd = 3.0e38f;
    constexpr int RUNS = CP_REGION_LIST / WAVE;
    float2 ce[RUNS];
    float de[RUNS];
#pragma unroll
    for (int u = 0; u < RUNS; ++u) ce[u] = reg_c[u * WAVE + lane < n_reg ? u * WAVE + lane : 0];
#pragma unroll
    for (int u = 0; u < RUNS; ++u) {
        de[u] = cells_dist2(mx, my, ce[u]);
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
        const bool k = u * WAVE + lane < n_reg && !cells_dominated(ce[u], de[u], nc, nd, w);
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
    mx = ((float)ix - 0.5f * G) * h;
    my = ((float)iy - 0.5f * G) * h;
    w = 0.5f * h + slack;
    const int quarter = (n_blk + 3) >> 2, e_begin = part * quarter, e_end = min(n_blk, e_begin + quarter);
    float da = 3.0e38f, db = 3.0e38f;                           // nearest and second nearest
    float2 ca = make_float2(0.0f, 0.0f), cb = ca;
    for (int e0 = e_begin; e0 < e_end; e0 += 4) {
        float2 c4[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) c4[q] = blk_c[wid][min(e0 + q, e_end - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float d = e0 + q < e_end ? cells_dist2(mx, my, c4[q]) : 3.0e38f;
            const bool first_of_all = d < da, second = d < db;
            cb.x = first_of_all ? ca.x : second ? c4[q].x : cb.x;
            cb.y = first_of_all ? ca.y : second ? c4[q].y : cb.y;
            db = first_of_all ? da : second ? d : db;
            ca.x = first_of_all ? c4[q].x : ca.x;
            ca.y = first_of_all ? c4[q].y : ca.y;
            da = first_of_all ? d : da;
        }
    }
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
    for (int e0 = e_begin; e0 < e_end; e0 += 4) {
        float2 c4[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) c4[q] = blk_c[wid][min(e0 + q, e_end - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float d = cells_dist2(mx, my, c4[q]);
            const bool out = cells_dominated(c4[q], d, ca, da, w) || (db < 3.0e38f && cells_dominated(c4[q], d, cb, db, w));
            if (!out && e0 + q < e_end) kept |= 1u << (e0 + q - e_begin);
        }
    }
    const int mine = __popc(kept);
    const int n0 = dpp_move<dpp_quad_lane(0)>(mine), n1 = dpp_move<dpp_quad_lane(1)>(mine), n2 = dpp_move<dpp_quad_lane(2)>(mine);
    int before = (part > 0 ? n0 : 0) + (part > 1 ? n1 : 0) + (part > 2 ? n2 : 0);
    const int total = n0 + n1 + n2 + dpp_move<dpp_quad_lane(3)>(mine);
    while (kept) {
        const int e = e_begin + __ffs((int)kept) - 1;
        kept &= kept - 1u;
        if (before < CELLS_LIST) rec_i[wid][cell][before] = blk_i[wid][e];
        ++before;
    }
    __syncthreads();
    if (part == 0) {
        uint2 r = make_uint2(0u, CELLS_SCAN);
        // the border belongs to everything outside the square: the lookup clamps to it
        const bool inside = ix > 0 && ix < G - 1 && iy > 0 && iy < G - 1;
        if (inside && total >= 1 && total <= CELLS_LIST) {
            unsigned i5[CELLS_LIST];
#pragma unroll
            for (int q = 0; q < CELLS_LIST; ++q) i5[q] = rec_i[wid][cell][q < total ? q : 0];
            // ascending; bits 3, 15, 27, 39, 51 onwards, padded with the first
            r.x = (i5[0] << 3) | (i5[1] << 15) | (i5[2] << 27) | (total > 3 ? CELLS_MORE : 0u);
            r.y = (i5[2] >> 5) | (i5[3] << 7) | (i5[4] << 19);
        }
        table[iy * G + ix] = r;
    }
}


// ------------------------------------------------------------------------------------------------ the search
// Byte offset, from 8 times `base`, of the record of the cell that holds (x0, x1).  The lookup rounds x G / 8 + G / 2 to the
// nearest integer and clamps it to the border, whose records say "whole codebook".
constexpr uint32_t CELLS_MAGIC_BITS = 0x4B000000u;             // 2^23: adding it rounds to an integer, left in the low bits
template <int G> __device__ __forceinline__ uint32_t cells_record_at(float x0, float x1, uint32_t table_at) {
    constexpr float inv_h = G / (2.0f * CELLS_HALF);
    constexpr float magic = 8388608.0f;
    const float vx = fminf(fmaxf(__builtin_fmaf(x0, inv_h, magic + G / 2), magic), magic + (G - 1));
    const float vy = fminf(fmaxf(__builtin_fmaf(x1, inv_h, magic + G / 2), magic), magic + (G - 1));
    // (iy G + ix) 8 + table_at mod 2^32, the two numbers' exponent bits taken out with the one constant
    const uint32_t cell = __float_as_uint(vy) * G + __float_as_uint(vx);
    return (cell << 3) + (table_at - ((CELLS_MAGIC_BITS * G + CELLS_MAGIC_BITS) << 3));
}
__device__ __forceinline__ bool cells_scan(uint2 rec) { return rec.y >> 31; }
// The nearest of the record's candidates, as its byte offset in the codebook (LDS, at byte address cb_at); m: its squared
// distance.  All lanes of the wave call it together.  FIVE: nearly every wave holds a pair with more than three candidates.
template <bool FIVE> __device__ __forceinline__ unsigned cells_nearest(uint2 rec, float x0, float x1, uint32_t cb_at, float &m) {
    const unsigned lo = rec.x, hi = rec.y;
    const unsigned o0 = lo & 0x7ff8u, o1 = (lo >> 12) & 0x7ff8u, o2 = __builtin_amdgcn_alignbit(hi, lo, 24) & 0x7ff8u;
    auto dist = [&](unsigned o) {
        const lds_f32x2_t c = lds_read<lds_f32x2_t>(cb_at + o);
        return exact_dist2(x0, x1, make_float2(c[0], c[1]));
    };
    const float d0 = dist(o0), d1 = dist(o1), d2 = dist(o2);
    m = fminf(fminf(d0, d1), d2);
    unsigned o = o2;
    if (FIVE || __ballot(lo & CELLS_MORE)) {
        const unsigned o3 = (hi >> 4) & 0x7ff8u, o4 = (hi >> 16) & 0x7ff8u;
        const float d3 = dist(o3), d4 = dist(o4);
        m = fminf(fminf(m, d3), d4);
        o = (d3 == m) ? o3 : o4;
        o = (d2 == m) ? o2 : o;
    }
    o = (d1 == m) ? o1 : o;                                     // the lowest index among equals: the candidates ascend
    return (d0 == m) ? o0 : o;
}

}  // namespace qamw
