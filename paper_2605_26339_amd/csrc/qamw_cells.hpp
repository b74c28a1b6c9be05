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
// all pairs (2^11 points, G = 128: 3.1 candidates on average over the pairs, never more than 5).  The lists are found
// top down -- 8 x 8 cells, 4 x 4 cells, single cells -- and each level searches only its parent's list.
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

// Candidate lists of 8 x 8 cells by one workgroup; wave w takes their w-th quarter of 4 x 4 cells.
template <int G>
__device__ __forceinline__ void cells_build_region(const float *codebook, int K, uint2 *table, int region) {
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
    float mx = ((float)x0 + 3.5f - 0.5f * G) * h, my = ((float)y0 + 3.5f - 0.5f * G) * h, w = 4.0f * h + slack;
    float nd = 3.0e38f;
    float2 nc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) {
        const bool have = j < per && first + j < K;
        c[j] = cbk[have ? first + j : 0];
        d2[j] = cells_dist2(mx, my, c[j]);
        if (d2[j] < nd) {
            nd = d2[j];
            nc = c[j];
        }
    }
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) {
        const float od = __shfl_xor(nd, s, WAVE), ox = __shfl_xor(nc.x, s, WAVE), oy = __shfl_xor(nc.y, s, WAVE);
        if (od < nd) {
            nd = od;
            nc = make_float2(ox, oy);
        }
    }
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
    for (int s = 1; s < WAVE; s <<= 1) {
        const int o = __shfl_up(below, s, WAVE);
        if (lane >= s) below += o;
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
    for (int e = lane; e < n_reg; e += WAVE) {
        const float2 ce = reg_c[e];
        const float d = cells_dist2(mx, my, ce);
        if (d < nd) {
            nd = d;
            nc = ce;
        }
    }
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) {
        const float od = __shfl_xor(nd, s, WAVE), ox = __shfl_xor(nc.x, s, WAVE), oy = __shfl_xor(nc.y, s, WAVE);
        if (od < nd) {
            nd = od;
            nc = make_float2(ox, oy);
        }
    }
    int n_blk = 0;
    for (int e0 = 0; e0 < n_reg; e0 += WAVE) {
        const int e = e0 + lane;
        const float2 ce = reg_c[e < n_reg ? e : 0];
        const bool k = e < n_reg && !cells_dominated(ce, cells_dist2(mx, my, ce), nc, nd, w);
        const unsigned long long mask = __ballot(k);
        const int pos = n_blk + __popcll(mask & ((1ull << lane) - 1ull));
        if (k && pos < CP_BLOCK_LIST) {
            blk_c[wid][pos] = ce;
            blk_i[wid][pos] = reg_i[e];
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
    for (int e = e_begin; e < e_end; ++e) {
        const float2 ce = blk_c[wid][e];
        const float d = cells_dist2(mx, my, ce);
        if (d < da) {
            db = da;
            cb = ca;
            da = d;
            ca = ce;
        } else if (d < db) {
            db = d;
            cb = ce;
        }
    }
#pragma unroll
    for (int s = 1; s <= 2; s <<= 1) {
        const float oda = __shfl_xor(da, s, WAVE), odb = __shfl_xor(db, s, WAVE);
        const float2 oca = make_float2(__shfl_xor(ca.x, s, WAVE), __shfl_xor(ca.y, s, WAVE));
        const float2 ocb = make_float2(__shfl_xor(cb.x, s, WAVE), __shfl_xor(cb.y, s, WAVE));
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
    }
    unsigned kept = 0;                                          // bit e - e_begin (a quarter is at most 32 candidates)
    for (int e = e_begin; e < e_end; ++e) {
        const float2 ce = blk_c[wid][e];
        const float d = cells_dist2(mx, my, ce);
        const bool out = cells_dominated(ce, d, ca, da, w) || (db < 3.0e38f && cells_dominated(ce, d, cb, db, w));
        if (!out) kept |= 1u << (e - e_begin);
    }
    const int mine = __popc(kept);
    int before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int o = __shfl(mine, (lane & ~3) | q, WAVE);
        if (q < part) before += o;
        total += o;
    }
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
// The record of the cell that holds (x0, x1): table in LDS.  The lookup rounds x G / 8 + G / 2 to the nearest integer and
// clamps it to the border, whose records say "whole codebook".
template <int G> __device__ __forceinline__ uint2 cells_record(const char *table, float x0, float x1) {
    constexpr float inv_h = G / (2.0f * CELLS_HALF);
    constexpr float magic = 8388608.0f;                        // 2^23: adding it rounds to an integer, left in the low bits
    const float vx = fminf(fmaxf(__builtin_fmaf(x0, inv_h, magic + G / 2), magic), magic + (G - 1));
    const float vy = fminf(fmaxf(__builtin_fmaf(x1, inv_h, magic + G / 2), magic), magic + (G - 1));
    const unsigned at = (__float_as_uint(vy) & 0xffffu) * (G * 8) + (__float_as_uint(vx) & 0xffffu) * 8;
    return *reinterpret_cast<const uint2 *>(table + at);
}
__device__ __forceinline__ bool cells_scan(uint2 rec) { return rec.y >> 31; }
// The nearest of the record's candidates, as its byte offset in the codebook (LDS); m: its squared distance.  All lanes of
// the wave call it together.  FIVE: nearly every wave holds a pair with more than three candidates.
template <bool FIVE> __device__ __forceinline__ unsigned cells_nearest(uint2 rec, float x0, float x1, const float2 *cb, float &m) {
    const unsigned lo = rec.x, hi = rec.y;
    const unsigned o0 = lo & 0x7ff8u, o1 = (lo >> 12) & 0x7ff8u, o2 = __builtin_amdgcn_alignbit(hi, lo, 24) & 0x7ff8u;
    auto dist = [&](unsigned o) {
        return exact_dist2(x0, x1, *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(cb) + o));
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
