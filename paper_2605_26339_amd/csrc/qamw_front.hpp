// Encoder front half shared by the fast encode and calibration kernels (Sec. 3.1 steps 1-2 on
// the channel-scaled row of Sec. B.2): a lane loads its 16 consecutive columns, scales them,
// divides by the row norm, applies the sign mask and the wave runs the block Walsh-Hadamard
// transform.  On return y[e] = (F S u)[col0 + e] exactly as the library's fp32 arithmetic defines it.
#pragma once
#include "qamw_common.hpp"
#include "qamw_internal.hpp"
#include "qamw_wave_fwht.hpp"

namespace qamw {

// The lane's 16 weights as loaded: 16 fp32 (DTYPE 0) or 16 bf16 in 8 dwords (DTYPE 1).  Split from the arithmetic so that
// a kernel can request the next row before it works on the current one.
template <int DTYPE> struct RawRow {
    uint32_t w[DTYPE == 0 ? 16 : 8];
};
template <int DTYPE>
__device__ __forceinline__ void load_raw_row(RawRow<DTYPE> &raw, const void *__restrict__ W, int64_t row_base, int c) {
    const int64_t base = row_base + c;
    if (DTYPE == 0) {
        const uint4 *w4 = reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(W) + base);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint4 v = w4[t];
            raw.w[4 * t] = v.x; raw.w[4 * t + 1] = v.y; raw.w[4 * t + 2] = v.z; raw.w[4 * t + 3] = v.w;
        }
    } else {
        const uint4 *w4 = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(W) + base);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint4 v = w4[t];
            raw.w[4 * t] = v.x; raw.w[4 * t + 1] = v.y; raw.w[4 * t + 2] = v.z; raw.w[4 * t + 3] = v.w;
        }
    }
}

// The 16 weights as fp32 (bf16 is the upper half of an fp32).
template <int DTYPE> __device__ __forceinline__ void widen_raw_row(float (&y)[16], const RawRow<DTYPE> &raw) {
    if (DTYPE == 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) y[e] = __uint_as_float(raw.w[e]);
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            y[2 * q] = __uint_as_float(raw.w[q] << 16);
            y[2 * q + 1] = __uint_as_float(raw.w[q] & 0xFFFF0000u);
        }
    }
}

// The scaled weights divided by the row's norm, which is the same in the whole wave; a zero norm gives zeros.
__device__ __forceinline__ void divide_by_norm(float (&y)[16], float norm) {
    // u = ws / r, the correctly rounded quotient.  With q = fl(1/r) correctly rounded, q0 = fl(ws q) and the exact
    // remainder rem = ws - q0 r (one fused multiply-add), fl(q0 + rem q) IS the correctly rounded ws / r (Markstein's
    // division theorem) as long as nothing under- or overflows on the way: r within 2^+-60 and every |ws| at least
    // 2^-100.  A wave that holds anything else (an exact zero included) takes the plain division for all its lanes.
    // (No value is set before the branches: zeros for a norm of zero, set there, were 16 moves in every row.)
    const uint32_t rb = __builtin_amdgcn_readfirstlane(__float_as_uint(norm));
    const float r = __uint_as_float(rb);
    float amin = fminf(fabsf(y[0]), fabsf(y[1]));
#pragma unroll
    for (int e = 2; e < 16; e += 2) amin = fminf(amin, fminf(fabsf(y[e]), fabsf(y[e + 1])));
    const bool usual = rb - 0x21800000u <= 0x5D800000u - 0x21800000u && __ballot(!(amin >= 0x1p-100f)) == 0ull;
    if (__builtin_expect(usual, true)) {
        // 1/r by the steps of the IEEE division; its scaling and its special cases do not arise
        const float e0 = __builtin_amdgcn_rcpf(r), e1 = __builtin_fmaf(__builtin_fmaf(-r, e0, 1.0f), e0, e0);
        const float e2 = __builtin_fmaf(__builtin_fmaf(-r, e1, 1.0f), e1, e1);
        const float q = __builtin_fmaf(__builtin_fmaf(-r, e2, 1.0f), e1, e2);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float q0 = y[e] * q;
            const float rem = __builtin_fmaf(-q0, r, y[e]);
            y[e] = __builtin_fmaf(rem, q, q0);
        }
    } else if (r > 0.0f) {
#pragma unroll
        for (int e = 0; e < 16; ++e) y[e] = y[e] / r;                           // IEEE division
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) y[e] = 0.0f;
    }
}

// c: first of the lane's 16 columns (multiple of 16, < d_in); r: the row's norm.
// Requires 16-byte aligned rows and side arrays (checked on the host).
template <int DTYPE, int B>
__device__ __forceinline__ void rotated_unit_row_from(float (&y)[16], const RawRow<DTYPE> &raw, int c, float r, const Problem &p,
                                                      const LaneSigns<B> &ls) {
    widen_raw_row<DTYPE>(y, raw);
    if (p.chan_scale) {
        const float4 *s4 = reinterpret_cast<const float4 *>(p.chan_scale + c);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float4 v = s4[t];
            y[4 * t] *= v.x; y[4 * t + 1] *= v.y; y[4 * t + 2] *= v.z; y[4 * t + 3] *= v.w;
        }
    }
    divide_by_norm(y, r);
    if (p.signs) {
        const uint4 sg = *reinterpret_cast<const uint4 *>(p.signs + c);
        const uint32_t wds[4] = {sg.x, sg.y, sg.z, sg.w};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            uint32_t neg = (wds[e >> 2] >> (8 * (e & 3) + 7)) & 1u;             // int8 -1: sign bit of the byte
            y[e] = __uint_as_float(__float_as_uint(y[e]) ^ (neg << 31));
        }
    }
    fwht_wave<B>(y, ls);
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = (y[e] * ls.parity) * p.inv_sqrt_block;
}

template <int DTYPE, int B>
__device__ __forceinline__ void rotated_unit_row(float (&y)[16], const void *__restrict__ W, int64_t row_base, int c,
                                                 float r, const Problem &p, const LaneSigns<B> &ls) {
    RawRow<DTYPE> raw;
    load_raw_row<DTYPE>(raw, W, row_base, c);
    rotated_unit_row_from<DTYPE, B>(y, raw, c, r, p, ls);
}

// ---------------------------------------------------------------------------------------------
// Row norms inside the kernels that need them (Sec. 3.1 step 1 on the channel-scaled row of Sec. B.2), so that the
// matrix is fetched from memory once per entry point instead of once by a norm kernel and once more by the kernel
// proper.
//
// A workgroup of NWAVES waves owns NWAVES consecutive (row, slab) items, which touch a few consecutive rows.  For every
// slab of every such row one wave sums the squares of the slab's 1024 scaled weights in fp64 (products of fp32 are
// exact in fp64; 16 per lane in column order, then the fixed butterfly of wave_sum) and leaves the sum in LDS; after
// the workgroup's barrier every wave adds its row's slab sums in slab order and takes the square root.  The value of a
// row's norm therefore does not depend on which workgroup computes it.  Rows shared by neighbouring workgroups are
// summed by each of them; fused_norm_block() numbers the workgroups so that neighbours run on the same XCD and
// find each other's rows in its L2.
// ---------------------------------------------------------------------------------------------
constexpr int FUSED_NORM_MAX_SLABS = 64;                       // rows of up to 65536 columns
constexpr int FUSED_NORM_XCDS = 8;

// Hardware workgroup b runs on XCD b mod 8.  Workgroup number used by the kernel: XCD x takes the x-th eighth of the
// work, in order.  A value >= n_blocks means: nothing to do.
__device__ __forceinline__ int fused_norm_block(int b, int n_blocks) {
    const int per = (n_blocks + FUSED_NORM_XCDS - 1) / FUSED_NORM_XCDS;
    return (b % FUSED_NORM_XCDS) * per + b / FUSED_NORM_XCDS;
}
inline int fused_norm_grid(int n_blocks) {                       // workgroups to launch for n_blocks of work
    return (n_blocks + FUSED_NORM_XCDS - 1) / FUSED_NORM_XCDS * FUSED_NORM_XCDS;
}

// acc + w^2: the square of an fp32 value is exact in fp64, so one rounding and the bits of a product and a sum.
__device__ __forceinline__ double add_square(double acc, float w) { return __builtin_fma((double)w, (double)w, acc); }

// Sum of squares of the scaled weights of columns [1024 slab, 1024 slab + 1024) of one row, the same in every lane.
template <int DTYPE>
__device__ __forceinline__ double slab_sum_of_squares(const void *__restrict__ W, int64_t row_base, int slab, const Problem &p,
                                                       int lane) {
    const int c = slab * 1024 + 16 * lane;
    double acc = 0.0;
    if (c < p.d_in) {
        RawRow<DTYPE> raw;
        load_raw_row<DTYPE>(raw, W, row_base, c);
        float w[16];
        if (DTYPE == 0) {
#pragma unroll
            for (int e = 0; e < 16; ++e) w[e] = __uint_as_float(raw.w[e]);
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                w[2 * q] = __uint_as_float(raw.w[q] << 16);
                w[2 * q + 1] = __uint_as_float(raw.w[q] & 0xFFFF0000u);
            }
        }
        if (p.chan_scale) {
            const float4 *s4 = reinterpret_cast<const float4 *>(p.chan_scale + c);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float4 v = s4[t];
                w[4 * t] *= v.x; w[4 * t + 1] *= v.y; w[4 * t + 2] *= v.z; w[4 * t + 3] *= v.w;
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) acc = add_square(acc, w[e]);
    }
    return wave_sum(acc);
}

// Slab sums of every row touched by the items [item0, item0 + NWAVES) (clipped to n_items) into part[], dealt to
// the workgroup's waves.  The caller's barrier follows; then row_norm_from_slab_sums().
// part: LDS, 2 * max(n_slabs, NWAVES) doubles.  All waves of the workgroup call this.
template <int DTYPE, int NWAVES>
__device__ __forceinline__ void block_slab_sums(double *part, const void *__restrict__ W, int64_t ldw, const Problem &p, int item0,
                                                int n_items, int n_slabs, int lane, int wid) {
    const int last = min(item0 + NWAVES, n_items) - 1;
    const int r0 = item0 / n_slabs, r1 = last / n_slabs;
    const int tasks = (r1 - r0 + 1) * n_slabs;
    for (int t = __builtin_amdgcn_readfirstlane(wid); t < tasks; t += NWAVES) {
        const int dr = t / n_slabs, slab = t - dr * n_slabs;
        const double s2 = slab_sum_of_squares<DTYPE>(W, (int64_t)(r0 + dr) * ldw, slab, p, lane);
        if (lane == 0) part[t] = s2;
    }
}

// The norm of `row` from the slab sums left by block_slab_sums() (after the barrier): slab order, fp64, one rounding
// to fp32 after the square root.
__device__ __forceinline__ float row_norm_from_slab_sums(const double *part, int row, int item0, int n_slabs) {
    const double *src = part + (row - item0 / n_slabs) * n_slabs;
    double s2 = 0.0;
    for (int s = 0; s < n_slabs; ++s) s2 += src[s];
    return (float)sqrt(s2);
}

// Sums of squares of R consecutive rows' scaled weights, by one wave: 16-byte loads, squares exact in fp64, the lane-strided
// sums combined with the fixed butterfly of wave_sum().  The same in every lane, and the same whatever R is.  n_rows <= R
// rows exist.  The scales are fetched once for the R rows.
template <int DTYPE, int R, bool SCALED>
__device__ __forceinline__ void wave_rows_sum_of_squares_as(double (&sum)[R], const void *__restrict__ W, int row, int n_rows, int64_t ldw,
                                                            int d_in, const float *__restrict__ s, int lane) {
    constexpr int V = DTYPE == 0 ? 4 : 8;                       // elements per 16-byte load
    constexpr int U = R == 1 ? 4 : 2;                           // loads per row requested together: a wave alone on its row has
                                                                // nothing else to hide the memory round trip behind
    const char *base[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        base[r] = reinterpret_cast<const char *>(W) + (int64_t)(row + (r < n_rows ? r : 0)) * ldw * (DTYPE == 0 ? 4 : 2);
        sum[r] = 0.0;
    }
    for (int j0 = lane * V; j0 < d_in; j0 += U * WAVE * V) {
        uint4 raw[R][U];
        float4 sv[U][V / 4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // past the end: the row's start again, taken as zeros (a branch would let the compiler move a load behind the sums
            // of those before it, one round trip each)
            const int j = j0 + u * WAVE * V, at = j < d_in ? j : 0;
#pragma unroll
            for (int r = 0; r < R; ++r) raw[r][u] = *reinterpret_cast<const uint4 *>(base[r] + (int64_t)at * (DTYPE == 0 ? 4 : 2));
            if (SCALED) {
#pragma unroll
                for (int t = 0; t < V / 4; ++t) sv[u][t] = *reinterpret_cast<const float4 *>(s + at + 4 * t);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t mask = j0 + u * WAVE * V < d_in ? 0xFFFFFFFFu : 0u;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float w[V];
                const uint32_t q4[4] = {raw[r][u].x & mask, raw[r][u].y & mask, raw[r][u].z & mask, raw[r][u].w & mask};
                if (DTYPE == 0) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) w[q] = __uint_as_float(q4[q]);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        w[2 * q] = __uint_as_float(q4[q] << 16);
                        w[2 * q + 1] = __uint_as_float(q4[q] & 0xFFFF0000u);
                    }
                }
                if (SCALED) {
#pragma unroll
                    for (int t = 0; t < V / 4; ++t) {
                        w[4 * t] *= sv[u][t].x; w[4 * t + 1] *= sv[u][t].y; w[4 * t + 2] *= sv[u][t].z; w[4 * t + 3] *= sv[u][t].w;
                    }
                }
#pragma unroll
                for (int t = 0; t < V; ++t) sum[r] = add_square(sum[r], w[t]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) sum[r] = wave_sum(sum[r]);
}
// (Without scales a loop of its own: multiplying by 1 cost a lone wave on a long fp32 row a fifth of its time.)
template <int DTYPE, int R>
__device__ __forceinline__ void wave_rows_sum_of_squares(double (&sum)[R], const void *__restrict__ W, int row, int n_rows, int64_t ldw,
                                                         int d_in, const float *__restrict__ s, int lane) {
    if (s) wave_rows_sum_of_squares_as<DTYPE, R, true>(sum, W, row, n_rows, ldw, d_in, s, lane);
    else wave_rows_sum_of_squares_as<DTYPE, R, false>(sum, W, row, n_rows, ldw, d_in, s, lane);
}

// The same sums in the order of slab_sum_of_squares() and row_norm_from_slab_sums(): to the bit what the kernels that compute
// their own row norms get.  R is 1 or 4: row + r's sum in the lanes from 64 r / R on; four rows share the last two steps of
// their butterflies.
template <int DTYPE, int R>
__device__ __forceinline__ double wave_rows_slab_sums(const void *__restrict__ W, int row, int n_rows, int64_t ldw, int d_in,
                                                      const float *__restrict__ s, int lane) {
    constexpr int U = R == 1 ? 2 : 1;                           // slabs requested together
    static_assert(R == 1 || R == 4, "wave_sum or wave_sum_4");
    double sum = 0.0;
    for (int slab = 0; slab * 1024 < d_in; slab += U) {
        RawRow<DTYPE> raw[U][R];
        float sc[U][16];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = (slab + u) * 1024 + 16 * lane, at = c < d_in ? c : 0;
#pragma unroll
            for (int r = 0; r < R; ++r) load_raw_row<DTYPE>(raw[u][r], W, (int64_t)(row + (r < n_rows ? r : 0)) * ldw, at);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float4 v = s ? reinterpret_cast<const float4 *>(s + at)[t] : make_float4(1.0f, 1.0f, 1.0f, 1.0f);
                sc[u][4 * t] = v.x; sc[u][4 * t + 1] = v.y; sc[u][4 * t + 2] = v.z; sc[u][4 * t + 3] = v.w;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if ((slab + u) * 1024 >= d_in) break;
            const bool have = (slab + u) * 1024 + 16 * lane < d_in;
            double acc[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float w[16];
                widen_raw_row<DTYPE>(w, raw[u][r]);
                acc[r] = 0.0;
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[r] = add_square(acc[r], w[e] * sc[u][e]);
                acc[r] = have ? acc[r] : 0.0;
            }
            if constexpr (R == 4) sum += wave_sum_4(acc);
            else sum += wave_sum(acc[0]);
        }
    }
    return sum;
}

// x = h + m + l exactly, each piece with at most 8 significant bits (a bf16 value held as fp32).
__device__ __forceinline__ void split3(float x, uint32_t &h, uint32_t &m, uint32_t &l) {
    h = __float_as_uint(x) & 0xFFFF0000u;
    const float r1 = x - __uint_as_float(h);
    m = __float_as_uint(r1) & 0xFFFF0000u;
    const float r2 = r1 - __uint_as_float(m);
    l = __float_as_uint(r2) & 0xFFFF0000u;
}
// two bf16 (given as fp32 bit patterns with a zero low half) into one dword: `even` in the low half
__device__ __forceinline__ uint32_t pack2(uint32_t even, uint32_t odd) { return (even >> 16) | odd; }

// Exact squared distance as every encoder decides with it: fma(e1, e1, e0 * e0), e = x - c.
__device__ __forceinline__ float exact_dist2(float x0, float x1, float2 c) {
    const float e0 = x0 - c.x, e1 = x1 - c.y;
    return __builtin_fmaf(e1, e1, e0 * e0);
}

// The pruned search's table (layout: qamw_search_grid_build): the record of the cell that holds (x0, x1), the first one's for
// a point outside the square.
__device__ __forceinline__ int grid_cell(float x0, float x1, float inv_h, int G, bool &inside) {
    const float half_g = 0.5f * (float)G, g_f = (float)G;
    // clamped to [-1, G] before the conversion (a NaN becomes -1): outside the square either way
    const int ix = (int)floorf(fminf(fmaxf(__builtin_fmaf(x0, inv_h, half_g), -1.0f), g_f));
    const int iy = (int)floorf(fminf(fmaxf(__builtin_fmaf(x1, inv_h, half_g), -1.0f), g_f));
    inside = (unsigned)ix < (unsigned)G && (unsigned)iy < (unsigned)G;
    return inside ? iy * G + ix : 0;
}
// The nearest of a record's eight candidates, the lowest index on ties; overflow: the cell has more candidates than that.
template <typename F>
__device__ __forceinline__ unsigned grid_nearest(const uint4 &rec, float x0, float x1, unsigned kmask, bool &overflow, F codeword) {
    const unsigned cand[8] = {rec.x & 0xffffu, rec.x >> 16, rec.y & 0xffffu, rec.y >> 16, rec.z & 0xffffu, rec.z >> 16, rec.w & 0xffffu, rec.w >> 16};
    overflow = cand[7] == 0xffffu;
    float bd = 3.0e38f;
    unsigned bi = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const unsigned ci = cand[j] & kmask;                    // (the overflow mark stays inside the codebook)
        const float dd = exact_dist2(x0, x1, codeword(ci));
        if (dd < bd) {
            bd = dd;
            bi = ci;
        }
    }
    return bi;
}

// The nearest of the K codewords in LDS to the point (x0, x1) (the same in all lanes), found by the whole wave: lane l
// scans the codewords l, l + 64, ..., then a lexicographic (distance, index) reduction over the lanes; the lowest index
// wins a tie.  Every lane returns the index (0 if every distance is NaN).  codeword(k): from wherever the caller keeps them.
// K_FROM, K_TO: what the caller knows of K; the loops that it rules out are left out.
template <int K_FROM, int K_TO, typename F> __device__ __forceinline__ int wave_exact_scan_of(float x0, float x1, F codeword, int K, int lane) {
    // Codewords requested together: the scan is a chain of LDS latencies otherwise.  Where 0.065 % of the pairs came here, one in three
    // of a wave's 512-pair items (2^11 points, cells of one width; with the cells of now 0.001 %), 13824 x 5120, the whole encode call,
    // took 156 us one at a time, 137 so.
    constexpr int AHEAD = 8;
    float bd = 3.0e38f;
    int bi = 0x7fffffff;
    auto look = [&](float2 c, int k) {
        const float dd = exact_dist2(x0, x1, c);
        if (dd < bd) {
            bd = dd;
            bi = k;
        }
    };
    if (K_TO >= AHEAD * WAVE && (K_FROM >= AHEAD * WAVE || K >= AHEAD * WAVE)) {   // K is a power of two
#pragma unroll 1
        for (int k0 = 0; k0 < K; k0 += AHEAD * WAVE) {
            float2 c[AHEAD];
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) c[j] = codeword(k0 + lane + j * WAVE);
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) look(c[j], k0 + lane + j * WAVE);
        }
    } else {                                                    // no more of them than there are
#pragma unroll 1
        for (int k = lane; k < K; k += WAVE) look(codeword(k), k);
    }
    const float least = wave_min(bd);
    unsigned long long at = __ballot(bd == least);
    int best = 0x7fffffff;
    while (at) {
        const int l = __ffsll((long long)at) - 1;
        at &= at - 1;
        best = min(best, __builtin_amdgcn_readlane(bi, l));
    }
    return best == 0x7fffffff ? 0 : best;
}
template <int K_FROM = 1, int K_TO = 4096>
__device__ __forceinline__ int wave_exact_scan(float x0, float x1, const float2 *cb_lds, int K, int lane) {
    return wave_exact_scan_of<K_FROM, K_TO>(x0, x1, [&](int k) { return cb_lds[k]; }, K, lane);
}
// the codewords at LDS byte address cb_at
template <int K_FROM = 1, int K_TO = 4096>
__device__ __forceinline__ int wave_exact_scan(float x0, float x1, uint32_t cb_at, int K, int lane) {
    return wave_exact_scan_of<K_FROM, K_TO>(x0, x1, [&](int k) {
        const lds_f32x2_t c = lds_read<lds_f32x2_t>(cb_at + 8u * (uint32_t)k);
        return make_float2(c[0], c[1]);
    }, K, lane);
}

// The lane's 8 pair gains g_k = 1 / sigma_k (IEEE division), or sqrt(d_in) when no pair scales are given; c = first of
// the lane's 16 columns.
__device__ __forceinline__ void load_pair_gains(float (&g)[8], const Problem &p, int c) {
    if (p.pair_sigma) {
        const float4 *g4 = reinterpret_cast<const float4 *>(p.pair_sigma + (c >> 1));
        const float4 a = g4[0], b = g4[1];
        const float sg8[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = 1.0f / sg8[k];                         // IEEE division
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = p.g_default;
    }
}

// 1/sqrt(B) is a power of two: its product with a gain is exact, and one multiplication by that gives the bits of the definition's
// two, y = t / sqrt(B) and x = y g, unless y is below the smallest normal number, where it is rounded.
constexpr bool unit_exact(int B) { return B == 64 || B == 256 || B == 1024; }
// Up to this gain that is nothing to a pair's distances: such a y times the gain is below 2^-102, so that its square is 0, and so are
// those of its differences from codewords that it could still change (below 2^-76).  (A phase can depend on whether y is 0.)  Usual gains are sqrt(d_in) and some powers of two around.
constexpr float UNIT_EXACT_MAX_GAIN = 0x1p24f;
// A lane's gains times its sign (the butterflies' parity) and 1/sqrt(B); or, where a lane of the wave has a larger gain, times the
// sign alone and true: the wave multiplies by 1/sqrt(B) first.
__device__ __forceinline__ bool combine_gains(float (&g)[8], float parity, float inv_sqrt_block) {
    float most = g[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) most = fmaxf(most, g[k]);
    const bool two = __ballot(!(most <= UNIT_EXACT_MAX_GAIN)) != 0ull;
    const float unit = two ? parity : parity * inv_sqrt_block;
#pragma unroll
    for (int k = 0; k < 8; ++k) g[k] = unit * g[k];
    return two;
}

// The lane's 16 channel scales with the sign mask in the sign bit: what a kernel that stays on one slab of a matrix keeps
// instead of both.  Scaling by it is exact as regards the sign: rounding commutes with negation, and a quotient, a sum of
// squares or a smallest magnitude does not see it.
__device__ __forceinline__ void load_signed_scales(float (&sc)[16], const Problem &p, int c) {
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] = 1.0f;
    if (p.chan_scale) {
        const float4 *s4 = reinterpret_cast<const float4 *>(p.chan_scale + c);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float4 v = s4[t];
            sc[4 * t] = v.x; sc[4 * t + 1] = v.y; sc[4 * t + 2] = v.z; sc[4 * t + 3] = v.w;
        }
    }
    if (p.signs) {
        const uint4 sg = *reinterpret_cast<const uint4 *>(p.signs + c);
        const uint32_t wds[4] = {sg.x, sg.y, sg.z, sg.w};
#pragma unroll
        for (int e = 0; e < 16; ++e)                            // int8 -1: sign bit of the byte
            sc[e] = __uint_as_float(__float_as_uint(sc[e]) ^ (((wds[e >> 2] >> (8 * (e & 3) + 7)) & 1u) << 31));
    }
}

// Writes the lane's 8 indices into the row's bit stream: 8 fields of p.bits bits are exactly p.bits bytes, byte aligned
// at byte (c / 16) * bits of the row.  The lane that holds the row's last 16 columns (col0 + 16 == d_in) zeroes the
// padding bytes of the row.
__device__ __forceinline__ void store_packed_fields(uint8_t *__restrict__ packed, int row, int c, int col0,
                                                    const unsigned (&idx)[8], const Problem &p) {
    const int bits = p.bits;
    uint8_t *dst = packed + (int64_t)row * p.row_bytes + (int64_t)(c >> 4) * bits;
    unsigned __int128 acc = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) acc |= (unsigned __int128)idx[k] << (k * bits);
    for (int t = 0; t < bits; ++t) dst[t] = (uint8_t)(acc >> (8 * t));
    if (col0 + 16 == p.d_in) {
        const int64_t used = (int64_t)(p.d_in >> 4) * bits;
        uint8_t *rowp = packed + (int64_t)row * p.row_bytes;
        for (int64_t t = used; t < p.row_bytes; ++t) rowp[t] = 0;
    }
}

// The same with the bit count known to the compiler: the fields are put together two by two, these shifted into dwords, and the
// dwords stored as one or two unaligned groups and the one to three bytes that remain.
template <int BITS, int UP> __device__ __forceinline__ void store_fields_n(uint8_t *dst, const unsigned (&idx)[8]) {
    typedef uint32_t u32_a1_t __attribute__((aligned(1)));
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    typedef u32x2_t u32x2_a1_t __attribute__((aligned(1)));
    typedef uint16_t u16_a1_t __attribute__((aligned(1)));
    static_assert(2 * BITS + UP <= 32, "two fields in a dword");
    uint32_t w[(8 * BITS + 31) / 32 + 1];
#pragma unroll
    for (int q = 0; q < (8 * BITS + 31) / 32 + 1; ++q) w[q] = 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t two = idx[2 * k] | (idx[2 * k + 1] << BITS);
        const int bit = 2 * k * BITS, word = bit >> 5, off = bit & 31;
        w[word] |= off >= UP ? two << (off - UP) : two >> (UP - off);
        if (off + 2 * BITS > 32) w[word + 1] |= two >> (32 - off + UP);
    }
    int at = 0;
    if (BITS >= 8) {
        *reinterpret_cast<u32x2_a1_t *>(dst) = u32x2_t{w[0], w[1]};
        at = 8;
    } else if (BITS >= 4) {
        *reinterpret_cast<u32_a1_t *>(dst) = w[0];
        at = 4;
    }
    if (BITS - at >= 4) {
        *reinterpret_cast<u32_a1_t *>(dst + at) = w[at / 4];
        at += 4;
    }
    if (BITS - at >= 2) {
        *reinterpret_cast<u16_a1_t *>(dst + at) = (uint16_t)w[at / 4];
        if (BITS - at == 3) dst[at + 2] = (uint8_t)(w[at / 4] >> 16);
    } else if (BITS - at == 1) {
        dst[at] = (uint8_t)w[at / 4];
    }
}
// row: the row's packed bytes; c: first of the lane's 16 columns; idx: the indices times 2^UP.
template <int UP = 0>
__device__ __forceinline__ void store_fields(uint8_t *row, int64_t row_bytes, int d_in, int c, const unsigned (&idx)[8], int bits) {
    uint8_t *dst = row + (int64_t)(c >> 4) * bits;
    switch (bits) {
        case 1: store_fields_n<1, UP>(dst, idx); break;
        case 2: store_fields_n<2, UP>(dst, idx); break;
        case 3: store_fields_n<3, UP>(dst, idx); break;
        case 4: store_fields_n<4, UP>(dst, idx); break;
        case 5: store_fields_n<5, UP>(dst, idx); break;
        case 6: store_fields_n<6, UP>(dst, idx); break;
        case 7: store_fields_n<7, UP>(dst, idx); break;
        case 8: store_fields_n<8, UP>(dst, idx); break;
        case 9: store_fields_n<9, UP>(dst, idx); break;
        case 10: store_fields_n<10, UP>(dst, idx); break;
        case 11: store_fields_n<11, UP>(dst, idx); break;
        default: store_fields_n<12, UP>(dst, idx); break;
    }
    if (c + 16 == d_in)                                         // the lane with the row's last columns zeroes the padding
        for (int64_t t = (int64_t)(d_in >> 4) * bits; t < row_bytes; ++t) row[t] = 0;
}

// Host-side check of what the vector loads above assume.
inline bool front_alignment_ok(const void *W, int dtype, int64_t ldw, const Problem &p) {
    const int64_t row_align = dtype == 0 ? 4 : 8;
    return (ldw % row_align == 0) && ((reinterpret_cast<uintptr_t>(W) & 15) == 0) &&
           (((reinterpret_cast<uintptr_t>(p.chan_scale) | reinterpret_cast<uintptr_t>(p.signs) |
              reinterpret_cast<uintptr_t>(p.pair_sigma)) & 15) == 0);
}

}  // namespace qamw
