// Fused dequantise-and-multiply for a few activation rows, Y = X W^T with W the decoded matrix
// (the follow-up the paper names in its Limitations: a fused dequantization-matmul kernel).
//
// The decoder is linear in the codewords (Sec. 3.2, Sec. B.2):
//     w_i = r_i * D_s^-1 S F yhat_i,        yhat_i,k = sigma_k * c[idx_ik]   (pair k of row i)
// and F is symmetric, S and D_s diagonal, so for an activation row x
//     <w_i, x> = r_i * < yhat_i, F S D_s^-1 x > = r_i * sum_k < c[idx_ik], z_k >,
//     z = the pairs of  sigma (.) F S (x / s).
// The weights are never rotated back: the ACTIVATIONS are rotated once (m rows, d_in log b adds
// each), and each packed index then costs one codeword lookup and two multiply-adds per
// activation row.  HBM traffic is the packed matrix, B/8 bytes per pair, against 4 bytes per pair
// for a bf16 matrix.
//
// Kernels: k_rotate_x (one wave per activation row and 1024-column slab, the encoder's register
// transform) and k_qgemv: a workgroup of 4 waves owns up to 64 rows of one matrix; its work is cut
// into (1024-column slab, 8-row group) steps, slab-major, and each wave takes a quarter of them; a
// wave holds the current slab's z in registers (the group's packed words requested together); per row it unpacks 8 indices,
// gathers 8 codewords from the LDS codebook and multiply-adds them into per-row, per-lane
// accumulators.  After each group one transposing reduction (each step
// trades half of the live sums with the lane whose number differs in one bit, so 8 sums per lane end
// as one row total per lane) adds the group's totals to the wave's running totals in LDS; at the end
// the 4 waves' totals are summed in a fixed order, times r_i, and stored.  The row count per
// workgroup is chosen per matrix so that every wave of a launch walks about the same, small number of
// (slab, row group) steps (about 4): a product alone in a launch -- as a forward pass issues most of them --
// takes as long as one wave's chain of dependent loads.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "qamw_common.hpp"
#include "qamw_internal.hpp"
#include "qamw_wave_fwht.hpp"

namespace qamw {

constexpr int GV_THREADS = 256;
constexpr int GV_WAVES = GV_THREADS / WAVE;
constexpr int GV_SLAB = 1024;
constexpr int GV_RG = 8;                // rows per group: requested together, accumulated together
constexpr int GV_STEPS_PER_WG = 16;     // target number of (slab, 8-row group) steps per workgroup: 4 per wave
constexpr int GV_MIN_WGS = 256;         // a matrix is cut into at least this many workgroups when it has the rows
constexpr int GV_MAX_ROWS_PER_WG = 64;
constexpr int GV_AHEAD_MAX_WGS_2 = 512;        // two activation rows: launches of at most this many workgroups keep two steps' packed words in registers
constexpr int GV_SELF_ROTATE_MAX_WGS = 1024;   // launches of at most this many workgroups (and one or two activation rows) skip k_rotate_x
constexpr int GV_MAX_M = 8;                // activation rows of the vector-ALU kernel
constexpr int GM_MAX_M = 64;               // ... of the matrix-core kernel (QAMW_MATMUL_MAX_ROWS of the public header)
constexpr int GM_ROWS = 32;                // weight rows of a workgroup: one tile of the matrix instruction
constexpr int GM_HALF_TILE_MAX_WGS = 256;  // launches that would make at most this many 32-row workgroups use 16-row ones
constexpr int GM_WAVES = 8;                // waves of a workgroup: each takes every eighth chunk of the rows
constexpr int GM_THREADS = GM_WAVES * WAVE;
constexpr int GM_CHUNK = 256;              // columns of one step of a wave: 2 halves x 16 instructions x 8 columns

typedef uint32_t gv_u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t gv_u32x2_t __attribute__((ext_vector_type(2)));
typedef float gv_f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 gv_bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 gv_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float gv_f32x4_t __attribute__((ext_vector_type(4)));
typedef float gv_f32x16_t __attribute__((ext_vector_type(16)));

// One product of a batch, as the kernels see it.  Z and partial point into the caller's workspace.
struct GemvMat {
    const void *X;
    const uint8_t *packed;
    const float *norms, *chan_scale, *pair_sigma;
    const int8_t *signs;
    float *Z, *Y;
    int64_t ldx, ldy, row_bytes;
    int d_out, d_in, n_slabs;
    int rows_per_wg;                       // rows one workgroup takes: a multiple of GV_RG, at most GV_MAX_ROWS_PER_WG
    float sigma_default;                   // 1/sqrt(d_in), used when pair_sigma is NULL
    int tok_tiles;                         // wide kernel: activation rows of a workgroup, in 128s
};
// Work lists of one launch: rotation items (activation row, slab) and workgroups (rows_per_wg rows), each numbered
// matrix-major.
struct GemvBatch {
    GemvMat mat[QAMW_MATMUL_MAX_BATCH];
    int rot_begin[QAMW_MATMUL_MAX_BATCH + 1];
    int grp_begin[QAMW_MATMUL_MAX_BATCH + 1];
    int n, m, K;
    int xdtype;                            // element type of X: 0 fp32, 1 bf16
    int gm_rows;                           // matrix-core kernel: weight rows per workgroup, 32 (a whole tile) or 16 (its upper half unused)
    float inv_sqrt_block;
    const float *codebook;
};
// The matrix of work item u: begin[] past the last matrix holds the total, so no entry there counts.  All of it is one scalar
// load; a loop over the matrices was a round trip each.
__device__ __forceinline__ int gv_find(const int (&begin)[QAMW_MATMUL_MAX_BATCH + 1], int u) {
    int i = 0;
#pragma unroll
    for (int k = 1; k < QAMW_MATMUL_MAX_BATCH; ++k) i += u >= begin[k] ? 1 : 0;
    return i;
}

// Where the matrix-core kernel keeps 8 consecutive bf16 columns col .. col+7 (col a multiple of 8) of activation row tok:
// in the order its B operand is read -- [32-row tile][256-column chunk][half of the chunk][instruction 0..15][row in the
// tile][8 columns] -- so that the 32 lanes of a half-wave load 512 consecutive bytes.  In elements.
__device__ __forceinline__ int64_t gm_z_offset(int tok, int col, int d_in) {
    const int tile = tok >> 5, r = tok & 31, ch = col >> 8, within = col & 255, h = within >> 7, j = (within & 127) >> 3;
    return ((((int64_t)tile * (d_in >> 8) + ch) * 2 + h) * 16 + j) * 256 + r * 8;
}

// z = sigma (.) F S (x / s) of activation row tok for one 1024-column slab: lane l returns the 16 columns of sub-block
// slab_pos(l) (the order of the register transform); all 64 lanes of the wave call it together.  Lanes past the end of
// the row work on columns 0..15 (their blocks hold no lane that counts) and return values nobody uses.
// In two halves, so that a caller can have other memory requests on their way between the loads and the arithmetic.
template <int MT> struct GvRotIn {          // what one lane loads: 16 values of each of MT activation rows, as they lie in
    uint32_t x[MT][16], sign[4];            // memory (16 dwords of fp32 or 8 of bf16), and their columns' constants
    float scale[16], sigma[8];
};
// tok[t]: the activation row that goes into x[t].  XDTYPE: the element type, or 2: that of the launch; bf16 rows are then read
// twice over, as many dwords as of fp32, without a branch.
template <int XDTYPE, int MT>
__device__ __forceinline__ void gv_rotate_load(GvRotIn<MT> &in, const GemvBatch &bt, const GemvMat &M, const int (&tok)[MT], int slab, int lane) {
    const float *spare = bt.codebook;                           // 64 readable bytes
    const int xdtype = XDTYPE == 2 ? bt.xdtype : XDTYPE;
    const int col0 = slab * GV_SLAB + 16 * slab_pos(lane);
    const int c = col0 < M.d_in ? col0 : 0;
    typedef gv_u32x4_t u32x4_a1_t __attribute__((aligned(1)));   // the rows and the columns' constants may lie anywhere
    auto load = [](const void *at, int i) { return reinterpret_cast<const u32x4_a1_t *>(at)[i]; };
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const char *row = static_cast<const char *>(M.X) + ((int64_t)tok[t] * M.ldx + c) * (xdtype == 0 ? 4 : 2);
#pragma unroll
        for (int i = 0; i < (XDTYPE == 1 ? 2 : 4); ++i) {
            const gv_u32x4_t v = load(row, xdtype == 0 ? i : i & 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) in.x[t][4 * i + k] = v[k];
        }
    }
    // Without branches, so that all of it is requested at once: what the call leaves out is read from the codebook, and not used.
    const float *scale = M.chan_scale ? M.chan_scale + c : spare, *sigma = M.pair_sigma ? M.pair_sigma + (c >> 1) : spare;
    const void *sign = M.signs ? static_cast<const void *>(M.signs + c) : spare;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const gv_u32x4_t v = load(scale, i);
#pragma unroll
        for (int k = 0; k < 4; ++k) in.scale[4 * i + k] = __uint_as_float(v[k]);
    }
    const gv_u32x4_t sg = load(sign, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) in.sign[k] = sg[k];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const gv_u32x4_t v = load(sigma, i);
#pragma unroll
        for (int k = 0; k < 4; ++k) in.sigma[4 * i + k] = __uint_as_float(v[k]);
    }
}
// The arithmetic: x times the reciprocal of the channel scale (the decoder's reciprocal, one Newton step), the sign mask,
// the transform, and one factor per pair -- lane sign of the transform x 1/sqrt(b) x sigma.
template <int B, int MT>
__device__ __forceinline__ void gv_rotate_compute(float (&y)[16], const GvRotIn<MT> &in, int t, int xdtype, const GemvBatch &bt, const GemvMat &M, int lane) {
    const LaneSigns<B> ls(lane);
    if (xdtype == 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) y[e] = __uint_as_float(in.x[t][e]);
    } else {
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            y[e] = __uint_as_float(in.x[t][e >> 1] << 16);
            y[e + 1] = __uint_as_float(in.x[t][e >> 1] & 0xFFFF0000u);
        }
    }
    // (selections, no branches: a load used in one branch alone is moved there, behind all that was to go on beside it)
    const bool scaled = M.chan_scale != nullptr, given = M.pair_sigma != nullptr;
    const uint32_t negative = M.signs ? 0x80000000u : 0u;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        y[e] = y[e] * fast_recip(scaled ? in.scale[e] : 1.0f);
        y[e] = __uint_as_float(__float_as_uint(y[e]) ^ ((in.sign[e >> 2] << (24 - 8 * (e & 3))) & negative));   // a negative byte: the other sign
    }
    fwht_wave<B>(y, ls);
    const float k = ls.parity * bt.inv_sqrt_block;
    float g[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) g[q] = k * (given ? in.sigma[q] : M.sigma_default);
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = y[e] * g[e >> 1];
}
template <int XDTYPE, int B>
__device__ __forceinline__ void gv_rotate_slab(float (&y)[16], const GemvBatch &bt, const GemvMat &M, int tok, int slab, int lane) {
    GvRotIn<1> in;
    const int toks[1] = {tok};
    gv_rotate_load<XDTYPE, 1>(in, bt, M, toks, slab, lane);
    gv_rotate_compute<B, 1>(y, in, 0, XDTYPE, bt, M, lane);
}

// z = sigma (.) F S (x / s) for every activation row, fp32, row-major [m][d_in]: a wave per row and slab.
template <int XDTYPE, int B>
__global__ __launch_bounds__(GV_THREADS) void k_rotate_x(GemvBatch bt) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = threadIdx.x >> 6;
    const int item = __builtin_amdgcn_readfirstlane(blockIdx.x * GV_WAVES + wid);
    if (item >= bt.rot_begin[bt.n]) return;
    const int mi = gv_find(bt.rot_begin, item);
    const GemvMat &M = bt.mat[mi];
    const int local = item - bt.rot_begin[mi];
    const int n_slabs = M.n_slabs;
    const int tok = __builtin_amdgcn_readfirstlane(local / n_slabs), slab = __builtin_amdgcn_readfirstlane(local % n_slabs);
    const int d_in = M.d_in;
    const int col0 = slab * GV_SLAB + 16 * slab_pos(lane);
    float y[16];
    gv_rotate_slab<XDTYPE, B>(y, bt, M, tok, slab, lane);
    if (col0 < d_in) {
        float4 *dst = reinterpret_cast<float4 *>(M.Z + (int64_t)tok * d_in + col0);
#pragma unroll
        for (int t = 0; t < 4; ++t) dst[t] = make_float4(y[4 * t], y[4 * t + 1], y[4 * t + 2], y[4 * t + 3]);
    }
}

// The same rounded to bf16 (nearest even), in the order above: a workgroup takes 8 R activation rows of one slab, R a wave.
// TURN: in LDS they are turned, so that 128 R consecutive bytes go to memory, where a row by itself writes 16 bytes to each of 128
// places (1000 rows of 4096, R = 2: 11.5 -> 9.4 us); few rows are sooner written as they are (64 rows: 0.5 us).  Rows from m up
// to the next multiple of 32 are zeros.
template <int XDTYPE, int B, int R, bool TURN>
__global__ __launch_bounds__(GM_THREADS) void k_rotate_tile(GemvBatch bt) {
    constexpr int ROWS = 8 * R, PITCH = 16 * ROWS + 16;         // bytes of eight columns of all rows; the 16 spread the lanes over the banks
    __shared__ __align__(16) char turned[TURN ? GV_SLAB / 8 * PITCH : 16];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = blockIdx.x;
    const int mi = gv_find(bt.rot_begin, item);
    const GemvMat &M = bt.mat[mi];
    const int local = item - bt.rot_begin[mi], n_slabs = M.n_slabs;
    const int group = local / n_slabs, slab = local - group * n_slabs, row0 = group * ROWS;
    const int d_in = M.d_in, pos = slab_pos(lane);
    int toks[R];
#pragma unroll
    for (int t = 0; t < R; ++t) toks[t] = min(row0 + wid * R + t, bt.m - 1);
    GvRotIn<R> in;
    gv_rotate_load<XDTYPE, R>(in, bt, M, toks, slab, lane);
#pragma unroll
    for (int t = 0; t < R; ++t) {
        float y[16];
        gv_rotate_compute<B, R>(y, in, t, XDTYPE, bt, M, lane);
        uint32_t o[8];
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const gv_f32x2_t v = {y[e], y[e + 1]};
            o[e >> 1] = row0 + wid * R + t < bt.m ? __builtin_bit_cast(uint32_t, __builtin_convertvector(v, gv_bf16x2_t)) : 0u;
        }
        if (!TURN) {
            const int col = slab * GV_SLAB + 16 * pos;
            uint16_t *z = reinterpret_cast<uint16_t *>(M.Z) + gm_z_offset(row0 + wid * R + t, col, d_in);
            if (col < d_in) {                                   // the next eight columns are those of the next instruction
                *reinterpret_cast<uint4 *>(z) = make_uint4(o[0], o[1], o[2], o[3]);
                *reinterpret_cast<uint4 *>(z + 32 * 8) = make_uint4(o[4], o[5], o[6], o[7]);
            }
            continue;
        }
        char *dst = turned + 2 * pos * PITCH + 16 * (wid * R + t);
        *reinterpret_cast<uint4 *>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<uint4 *>(dst + PITCH) = make_uint4(o[4], o[5], o[6], o[7]);
    }
    if (!TURN) return;
    __syncthreads();
    uint16_t *zb = reinterpret_cast<uint16_t *>(M.Z);
#pragma unroll
    for (int i = threadIdx.x; i < GV_SLAB / 8 * ROWS; i += GM_THREADS) {
        const int j = i / ROWS, row = i % ROWS, col = slab * GV_SLAB + 8 * j;
        if (col < d_in) *reinterpret_cast<uint4 *>(zb + gm_z_offset(row0 + row, col, d_in)) = *reinterpret_cast<const uint4 *>(turned + j * PITCH + 16 * row);
    }
}

// Field i of a lane's stream as a byte offset into the codebook, index times 8: one shift and one AND, with the mask in a register
// (an AND of two registers issues at twice the rate of one with a literal).
//   Never a plain shift to the left by one or two: the compiler then takes the offset for a multiple of two or four, the mask being
// opaque, and reads the codeword as two halves, each with the bank conflicts of the whole (11 bits, one codeword in eight: 11008 x
// 4096, one row, 14.8 us by the trace, 14.0 so; 13824 x 5120 19.9, 18.9).
template <int BITS> __device__ __forceinline__ uint32_t gv_field_x8(const uint32_t (&w)[4], int i, uint32_t mask8) {
    const int bit = i * BITS, word = bit >> 5, off = bit & 31, s = off - 3;
    const uint32_t v = s == -3 ? w[word] << 3 : s < 0 ? __builtin_amdgcn_alignbit(w[word], w[word - 1], 32 + s) : off + BITS <= 32 ? w[word] >> s : __builtin_amdgcn_alignbit(w[word + 1], w[word], s);
    return v & mask8;
}

// Sums over the 64 lanes of N per-lane values a[0..N), N a power of two <= 64, leaving ONE total per lane:
// each step pairs lane l with lane l ^ 2^bit (bit = 5, 4, ..., ), every lane keeps the half of the live values
// selected by that bit of its number and adds what its partner held for that half.  When one value is left
// the remaining bits are summed in the ordinary way.  On return a[0] is the total of row gv_lane_row<N>(lane).
template <int N> __device__ __forceinline__ int gv_lane_row(int lane) {
    int row = 0, n = N;
#pragma unroll
    for (int bit = 5; bit >= 0 && n > 1; --bit) {
        n >>= 1;
        row += ((lane >> bit) & 1) * n;
    }
    return row;
}
// The value of the lane whose number differs in bit BIT, for bits 0 to 3 by DPP moves: a shuffle through LDS is some 120 cycles, four
// of them after another in every step of a wave.
template <int BIT> __device__ __forceinline__ float gv_xor_lane(float v) {
    if constexpr (BIT == 0) return dpp_move<DPP_XOR1>(v);
    else if constexpr (BIT == 1) return dpp_move<DPP_XOR2>(v);
    else if constexpr (BIT == 2) return dpp_move<DPP_QUAD_REVERSE>(dpp_move<DPP_HALF_MIRROR>(v));   // l ^ 7, then ^ 3
    else if constexpr (BIT == 3) return dpp_move<DPP_ROW_ROTATE_8>(v);
    else return __shfl_xor(v, 1 << BIT, WAVE);
}
// one step: LIVE values are live in a[0..LIVE); lane l pairs with lane l ^ 2^BIT
template <int N, int LIVE, int BIT> __device__ __forceinline__ void gv_reduce_step(float (&a)[N], int lane) {
    if constexpr (LIVE > 1) {
        constexpr int H = LIVE / 2;
#pragma unroll
        for (int r = 0; r < H; ++r) {
            if constexpr (BIT == 5) {
                auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[r]), __float_as_uint(a[r + H]), false, false);
                a[r] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            } else if constexpr (BIT == 4) {
                auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[r]), __float_as_uint(a[r + H]), false, false);
                a[r] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            } else {
                const bool up = (lane >> BIT) & 1;
                const float send = up ? a[r] : a[r + H], keep = up ? a[r + H] : a[r];
                a[r] = keep + gv_xor_lane<BIT>(send);
            }
        }
    } else {
        a[0] += gv_xor_lane<BIT>(a[0]);
    }
}
template <int N> __device__ __forceinline__ void gv_reduce_rows(float (&a)[N], int lane) {
    static_assert(N >= 1 && N <= 64 && (N & (N - 1)) == 0, "rows per reduction");
    gv_reduce_step<N, N, 5>(a, lane);
    gv_reduce_step<N, (N > 1 ? N / 2 : 1), 4>(a, lane);
    gv_reduce_step<N, (N > 2 ? N / 4 : 1), 3>(a, lane);
    gv_reduce_step<N, (N > 4 ? N / 8 : 1), 2>(a, lane);
    gv_reduce_step<N, (N > 8 ? N / 16 : 1), 1>(a, lane);
    gv_reduce_step<N, (N > 16 ? N / 32 : 1), 0>(a, lane);
}

// Y[t][row] = r_row * sum over the row's pairs of <c[idx], z_t>.  RB == 0: z comes from the workspace (k_rotate_x ran
// before).  RB > 0 (the block size): every wave rotates the slabs it needs itself, with the same arithmetic, and moves
// the result from the transform's lane order to the natural one -- the same z in the same lanes, so the same Y, bit for
// bit, without the first launch; for launches so small that a second launch costs more than the repeated rotations.
// AHEAD (self-rotating kernels only): the steps whose packed words the wave keeps in registers.  2: one activation row fits
// three waves per SIMD (768 resident workgroups: a launch of up to 1024 finishes its last quarter in a second round),
// two rows fit two (512 workgroups: the host picks the plain form for larger two-row launches).  1: no wave has a second step;
// requests for steps that there are not are answered with zeros, but take the address unit's time (one row at 11 bits, by the trace,
// with 2 / 1: 5632 x 2048 8.0 / 6.9 us, 1024 x 4096 6.7 / 5.6, 256 x 2048 6.4 / 5.5).
#define QAMW_GV_WAVES_PER_EU (AHEAD ? (MT == 1 ? 3 : 2) : 1)
template <int BITS, int MT, int RB, int AHEAD>
__global__ __launch_bounds__(GV_THREADS) __attribute__((amdgpu_waves_per_eu(QAMW_GV_WAVES_PER_EU)))
void k_qgemv(GemvBatch bt) {
    constexpr int RG = MT == 8 ? 4 : GV_RG, UR = GV_MAX_ROWS_PER_WG;
    // statically sized, so that a codeword's address is its index times 8 with nothing to add (bt.K == 2^BITS)
    __shared__ float2 cb_lds[1 << BITS];                        // the codewords
    __shared__ float red[GV_WAVES * UR * MT];                   // [waves][UR rows][MT]
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform over the wave: keeps the step bookkeeping scalar

    const int grp = blockIdx.x;                                 // the grid is exactly the number of workgroups
    const int mi = gv_find(bt.grp_begin, grp);
    const GemvMat M = bt.mat[mi];
    // All that the wave needs of the arguments is asked for here, in two round trips of scalar loads: what a branch or a later
    // use fetches for itself is one more each.
    asm volatile("" ::"s"(M.X), "s"(M.packed), "s"(M.norms), "s"(M.chan_scale), "s"(M.pair_sigma), "s"(M.signs), "s"(M.Y), "s"(M.ldx),
                 "s"(M.ldy), "s"(M.row_bytes), "s"(M.d_out), "s"(M.d_in), "s"(M.n_slabs), "s"(M.rows_per_wg), "s"(M.sigma_default),
                 "s"(bt.codebook), "s"(bt.m), "s"(bt.xdtype), "s"(bt.inv_sqrt_block), "s"(bt.grp_begin[mi]));
    const int rpw = M.rows_per_wg;
    const int row0 = (grp - bt.grp_begin[mi]) * rpw;
    const int n_g = rpw / RG;                                   // row groups of this workgroup
    const int n_slabs = M.n_slabs, m = bt.m;
    const int d_in = M.d_in, last_row = M.d_out - 1;
    int64_t row_bytes = M.row_bytes;
    const uint8_t *packed = M.packed;
    const float *Z = M.Z;

    auto lane_col = [&](int slab) __attribute__((always_inline)) {                             // first of the lane's 16 columns (0 for idle lanes)
        const int col0 = slab * GV_SLAB + 16 * lane;           // no transform here: lanes in natural column order
        return col0 < d_in ? col0 : 0;
    };
    // A lane's 8 fields are BITS bytes, at the same place in every row of a slab: 16 bytes from a 4-byte-aligned address hold
    // them, up to 16 - BITS of them the next row's.  Where that could be past the matrix's end -- in a group that reaches its
    // last row -- they are taken further to the front (field_shift() dwords), and rows past the end re-read the last row.
    auto last_group = [&](int r0) __attribute__((always_inline)) { return r0 + RG - 1 >= last_row; };
    auto field_at = [&](int slab) __attribute__((always_inline)) { return (unsigned)(lane_col(slab) >> 4) * BITS; };
    auto field_base = [&](int slab, int r0) __attribute__((always_inline)) {
        const unsigned at = field_at(slab) & ~3u;
        return last_group(r0) ? min(at, (unsigned)row_bytes - 16u) : at;
    };
    // The packed words of a group of rows.  Buffer loads without a branch: the compiler then knows how many are under way, and
    // waits for those that it needs, whatever comes after them.  wanted: otherwise the loads are out of range, read nothing and
    // give zeros.  (A group's rows lie within 2^31 bytes.)
    auto fetch = [&](int slab, int g, bool wanted, uint32_t (&d)[RG][4]) __attribute__((always_inline)) {
        const int r0 = min(row0 + g * RG, last_row);
        const unsigned at = field_base(slab, r0);
        const uint32_t rb = (uint32_t)row_bytes, most = wanted ? (uint32_t)min(last_row - r0, RG - 1) * rb : 0u;
        const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(packed + (int64_t)r0 * row_bytes), 0,
                                                            wanted ? (int)(most + rb + 16u) : 0, 0x00020000);
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            const gv_u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rows, at, min(r * rb, most), 0);
            d[r][0] = v[0]; d[r][1] = v[1]; d[r][2] = v[2]; d[r][3] = v[3];
        }
    };
    // the lane whose transform sub-block is this lane's natural one (slab_pos permutes inside groups of 16 lanes)
    int z_from = 0;
    if (RB > 0) {
#pragma unroll
        for (int l = 0; l < 16; ++l) z_from = (slab_pos(l) == (lane & 15)) ? l : z_from;
        z_from = ((lane & ~15) | z_from) << 2;
    }
    // The slab's rotated activations, zero for missing rows of X and idle lanes: the self-rotating kernels load the
    // inputs (rot_load) and rotate (rot_finish) in two steps, the others read the rotation kernel's output.
    auto rot_load = [&](int slab, GvRotIn<MT> &in) __attribute__((always_inline)) {
        int toks[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) toks[t] = t < m ? t : 0;
        gv_rotate_load<2, MT>(in, bt, M, toks, slab, lane);
    };
    auto rot_finish = [&](int slab, const GvRotIn<MT> &in, float (&z)[MT][16]) __attribute__((always_inline)) {
        const bool active = slab * GV_SLAB + 16 * lane < d_in;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const bool have = active && t < m;
            float y[16];
            constexpr int B = RB > 0 ? RB : 64;
            gv_rotate_compute<B, MT>(y, in, t, bt.xdtype, bt, M, lane);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float v = __int_as_float(__builtin_amdgcn_ds_bpermute(z_from, __float_as_int(y[e])));
                z[t][e] = have ? v : 0.0f;
            }
        }
    };
    auto load_z = [&](int slab, float (&z)[MT][16]) __attribute__((always_inline)) {
        if constexpr (RB > 0) {
            GvRotIn<MT> in;
            rot_load(slab, in);
            rot_finish(slab, in, z);
        } else {
            const bool active = slab * GV_SLAB + 16 * lane < d_in;
            const int c = lane_col(slab);
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const bool have = active && t < m;
                const float4 *src = reinterpret_cast<const float4 *>(Z + (int64_t)(t < m ? t : 0) * d_in + c);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 v = src[q];
                    z[t][4 * q] = have ? v.x : 0.0f;
                    z[t][4 * q + 1] = have ? v.y : 0.0f;
                    z[t][4 * q + 2] = have ? v.z : 0.0f;
                    z[t][4 * q + 3] = have ? v.w : 0.0f;
                }
            }
        }
    };

    constexpr int NORMS = (UR * MT + GV_THREADS - 1) / GV_THREADS;   // of the rows whose sums the thread stores: not a round trip at the end
    float norm[NORMS];
    auto load_norms = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NORMS; ++i) norm[i] = M.norms[min(row0 + ((int)threadIdx.x + i * GV_THREADS) / MT, last_row)];
    };

    // The workgroup's work is n_slabs x n_g steps (slab-major: one slab's row groups are consecutive); wave w takes
    // the w-th quarter of them, so the waves are equally loaded whatever the slab count is.
    const int n_steps = n_slabs * n_g;
    const int per_wave = (n_steps + GV_WAVES - 1) / GV_WAVES;
    int step0 = wid * per_wave;
    const int step1 = min(n_steps, step0 + per_wave);
    float z[MT][16];
    int cur_slab = min(step0, n_steps - 1) / n_g;
    const int my_row = gv_lane_row<RG>(lane);                   // after the reduction: which of the group's rows this lane holds
    float *my_red = red + wid * UR * MT;                        // this wave's running row totals (only this wave touches them until the last barrier)

    // one step: the group's 8 x 64 x 8 codeword gathers and multiply-adds, the totals over the lanes, into my_red
    // (once: no other step of the wave is of these rows)
    uint32_t mask8;                                             // ((1 << BITS) - 1) * 8 in a register the optimiser cannot fold back into a literal
    asm volatile("v_mov_b32 %0, %1" : "=v"(mask8) : "n"(((1 << BITS) - 1) * 8));
    auto work = [&](auto once, int slab, int g, uint32_t (&d)[RG][4]) __attribute__((always_inline)) {
        const int r0 = row0 + g * RG;
        const unsigned field = field_at(slab);
        const int sh = (int)(field & 3u) * 8;
        if (last_group(r0)) {                                   // words taken from further to the front
            const unsigned shift = (field & ~3u) - field_base(slab, r0);
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const uint32_t w1 = d[r][1], w2 = d[r][2], w3 = d[r][3];
                d[r][0] = shift == 0 ? d[r][0] : shift == 4 ? w1 : w2;
                d[r][1] = shift == 0 ? w1 : shift == 4 ? w2 : w3;
                d[r][2] = shift == 0 ? w2 : w3;
            }
        }
        float acc[MT][RG];
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int r = 0; r < RG; ++r) acc[t][r] = 0.0f;
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            uint32_t w[4];
            w[0] = __builtin_amdgcn_alignbit(d[r][1], d[r][0], sh);
            w[1] = __builtin_amdgcn_alignbit(d[r][2], d[r][1], sh);
            w[2] = __builtin_amdgcn_alignbit(d[r][3], d[r][2], sh);
            w[3] = d[r][3] >> sh;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float2 cw = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(cb_lds) + gv_field_x8<BITS>(w, k, mask8));
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    acc[t][r] = __builtin_fmaf(cw.y, z[t][2 * k + 1], __builtin_fmaf(cw.x, z[t][2 * k], acc[t][r]));
            }
        }
        // totals over the lanes: every lane ends with one of the group's RG rows (64 / RG lanes hold each, the ones that
        // share the lane number's upper bits); the first of them adds it in
#pragma unroll
        for (int t = 0; t < MT; ++t) gv_reduce_rows<RG>(acc[t], lane);
        if ((lane & (WAVE / RG - 1)) == 0) {
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                float &sum = my_red[(g * RG + my_row) * MT + t];
                sum = decltype(once)::value ? acc[t][0] : sum + acc[t][0];
            }
        }
    };
    struct Place {                                              // of a step
        int slab, g;
    };
    auto place = [&](int step) __attribute__((always_inline)) { return Place{step / n_g, step - step / n_g * n_g}; };
    auto advance = [&](Place &at) __attribute__((always_inline)) {
        if (++at.g == n_g) {
            at.g = 0;
            ++at.slab;
        }
    };

    static_assert(!AHEAD || RB > 0, "only the self-rotating kernels run ahead");
    if constexpr (!AHEAD) {
        load_z(cur_slab, z);                                    // on its way while the codebook is staged
        // For more than one activation row the codebook goes from memory straight into LDS: wave w copies the 1 KB
        // pieces w, w + 4, ..., lane l the 16 bytes l of a piece (the instruction places lane l's bytes at base + 16 l);
        // measured 6 % faster at m = 4, 1-3 % slower at m = 1, where it goes through registers.
        if (MT > 1) {
            const char *src = reinterpret_cast<const char *>(bt.codebook);
            const int bytes = bt.K * (int)sizeof(float2);
            for (int off = wid * 1024; off < bytes; off += GV_WAVES * 1024) {
                if (off + 16 * lane < bytes)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + off + 16 * lane),
                                                     (__attribute__((address_space(3))) void *)(reinterpret_cast<char *>(cb_lds) + off),
                                                     16, 0, 0);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): this wave's pieces have landed before the barrier
        } else {
            const float2 *cbk = reinterpret_cast<const float2 *>(bt.codebook);
            for (int i = threadIdx.x; i < bt.K; i += GV_THREADS) cb_lds[i] = cbk[i];
        }
        for (int i = lane; i < UR * MT; i += WAVE) my_red[i] = 0.0f;
        __syncthreads();
        load_norms();
#pragma unroll 1
        for (int step = step0; step < step1; ++step) {
            const Place at = place(step);
            if (at.slab != cur_slab) {
                load_z(at.slab, z);
                cur_slab = at.slab;
            }
            uint32_t d[RG][4];
            fetch(at.slab, at.g, true, d);
            work(std::false_type{}, at.slab, at.g, d);
        }
    } else {
        // A launch that rotates the activations itself is a small one -- one to three waves per SIMD, one to four steps
        // per wave -- and lasts as long as one wave's chain of memory round trips.  So the chain is kept short: the
        // rotation's inputs, the workgroup's share of the codebook, the packed words of the wave's first two steps (or its only one) and the norms
        // are requested before anything is waited for (the rotation's first: it has arithmetic to do while the rest
        // arrives), and from then on the next step's packed words are on their way while a step is worked on.  What stood in
        // the way: a branch on the element type or on the matrix's last row, at which the compiler waits for what either side
        // may have asked for, loads moved into the branch that uses them, a loop of scalar loads, the rotation inputs of a
        // wave's second and third slab.  A 7B layer's four launches, one row: 67 us, so 58; then issue-bound, 8 instructions
        // a codeword, where the launch has two waves and more per SIMD (11008 x 4096 twice: 19 us, 62 MB).
        // bt.K == 2^BITS here.
        constexpr int KC = 1 << BITS, CB_PER_THREAD = (KC + GV_THREADS - 1) / GV_THREADS;
        GvRotIn<MT> rin;
        rot_load(cur_slab, rin);
        // in this order, and the addresses of the packed words not worked out before it is their turn (0.5 us)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+s"(row_bytes));
        asm volatile("" : "+s"(step0));
        float2 cbv[CB_PER_THREAD];
        const float2 *cbk = reinterpret_cast<const float2 *>(bt.codebook);
#pragma unroll
        for (int j = 0; j < CB_PER_THREAD; ++j) cbv[j] = cbk[min((int)threadIdx.x + j * GV_THREADS, KC - 1)];
        __builtin_amdgcn_sched_barrier(0);
        uint32_t da[RG][4], db[RG][4];
        Place at = place(min(step0, n_steps - 1)), ask = at;
        auto fetch_next = [&](int step, uint32_t (&d)[RG][4]) __attribute__((always_inline)) {
            fetch(ask.slab, ask.g, step < step1, d);            // (past the wave's last step: places that may not exist, not read)
            advance(ask);
        };
        fetch_next(step0, da);
        if constexpr (AHEAD > 1) fetch_next(step0 + 1, db);
        load_norms();
        __builtin_amdgcn_sched_barrier(0);
        rot_finish(cur_slab, rin, z);
#pragma unroll
        for (int j = 0; j < CB_PER_THREAD; ++j)
            if ((int)threadIdx.x + j * GV_THREADS < KC) cb_lds[threadIdx.x + j * GV_THREADS] = cbv[j];
        for (int i = lane; i < UR * MT; i += WAVE) my_red[i] = 0.0f;
        __syncthreads();
        // SEVERAL: the wave's steps are of more than one slab.  The next one's rotation inputs are then asked for while a slab is
        // worked on (for one activation row: two rows' inputs would cost registers that are not there).
        const int last_slab = step0 < step1 ? (step1 - 1) / n_g : cur_slab;
        auto walk = [&](auto several) __attribute__((always_inline)) {
            constexpr bool SEVERAL = decltype(several)::value, EARLY = MT == 1;
            if (SEVERAL && EARLY) rot_load(cur_slab + 1, rin);
            auto next = [&](uint32_t (&d)[RG][4]) __attribute__((always_inline)) {
                if (SEVERAL && at.slab != cur_slab) {
                    if (!EARLY) rot_load(at.slab, rin);
                    rot_finish(at.slab, rin, z);
                    if (EARLY) rot_load(min(at.slab + 1, last_slab), rin);
                    cur_slab = at.slab;
                }
                work(std::bool_constant<!SEVERAL>{}, at.slab, at.g, d);
                advance(at);
            };
#pragma unroll 1
            for (int step = step0; step < step1; step += 2) {
                next(da);
                fetch_next(step + 2, da);
                if (step + 1 < step1) next(db);
                fetch_next(step + 3, db);
            }
        };
        if constexpr (AHEAD == 1) {
            if (step0 < step1) work(std::true_type{}, at.slab, at.g, da);
        } else if (last_slab > cur_slab) {
            walk(std::true_type{});
        } else {
            walk(std::false_type{});
        }
    }
    __syncthreads();
    // the 4 waves' sums in wave order, times the row norm
#pragma unroll
    for (int i = 0; i < NORMS; ++i) {
        const int o = threadIdx.x + i * GV_THREADS, row = o / MT, t = o - row * MT;
        if (o < rpw * MT && t < m && row0 + row <= last_row) {
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < GV_WAVES; ++w) s += red[(w * UR + row) * MT + t];
            M.Y[(int64_t)t * M.ldy + row0 + row] = norm[i] * s;
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// More than 8 activation rows: the products go to the bf16 matrix cores.
//   Y[t][i] = r_i * sum_k < bf16(c[idx_ik]), bf16(z_tk) >,   fp32 accumulation,
// z as above but rounded to bf16 (round to nearest even) by k_rotate_x, the codewords rounded to bf16 when the
// workgroup stages them: what a bf16 matmul on a bf16 copy of the rotated-domain operands computes.
//
// v_mfma_f32_32x32x16_bf16 with A = 32 weight rows x 16 columns, B = 16 columns x 32 activation rows: lane
// (r, h) supplies row r's 8 columns of half h to A -- exactly 4 pairs, i.e. 4 codewords, each one 32-bit
// LDS gather of (bf16 c0, bf16 c1) -- and activation row r's same 8 columns to B (16 bytes of z).
// A workgroup of 8 waves owns 32 weight rows (one tile); the 256-column chunks of the rows are dealt to the
// waves round-robin; within a chunk half h of the wave covers columns 128h .. 128h+127, so a lane walks 64
// consecutive pairs of its row: 8*BITS consecutive bytes, read as BITS 8-byte words from the wave's LDS copy
// of the chunk and unpacked at compile-time bit offsets.  No barrier inside the loop; the eight waves' tiles
// are summed through LDS in wave order at the end.  The shape follows from what bounds a launch: the chain of
// dependent chunk loads of its longest workgroup (a wave has one chunk in flight), so short chains -- many
// waves per row, few rows per workgroup -- beat shared operands; 128 registers keep 16 waves on a CU.
template <int BITS> __device__ __forceinline__ uint32_t gm_field_x4(const uint32_t (&w)[2 * BITS], int i) {
    // 4 * (field i of the lane's 64-field stream): the byte offset of the codeword in the bf16 table
    const int bit = i * BITS, word = bit >> 5, off = bit & 31;
    const uint32_t v = (off + BITS <= 32) ? (w[word] >> off) : __builtin_amdgcn_alignbit(w[word + 1], w[word], off);
    return (v & ((1u << BITS) - 1u)) << 2;
}

// ROWS: rows of the tile that a workgroup fills: all 32, or 16 (a launch of few workgroups is cut finer so that it covers the
// chip; a row's sum is the same chunks in the same waves in the same order either way, bit for bit).  The tile's other rows are
// then the same 16 again, gathers of the same addresses, and are not stored.
template <int BITS, int MT, int ROWS>
__global__ __launch_bounds__(GM_THREADS) __attribute__((amdgpu_waves_per_eu(4, 8)))   // two workgroups per CU: at most 128 registers
void k_qgemm(GemvBatch bt) {
    extern __shared__ __align__(16) uint32_t gm_lds[];
    uint32_t *cbh = gm_lds;                                     // K codewords as (bf16 c0) | (bf16 c1) << 16
    // after the codebook: per wave a 32-row tile of packed bytes (pitch PITCH) during the loop, and, after it, the
    // waves' partial tiles: [8 waves][32 activation rows][32 + 1 weight rows]
    float *red = reinterpret_cast<float *>(gm_lds + bt.K);
    constexpr int PITCH = 16 * BITS + 8;                        // bytes; an odd number of 8-byte words: the lanes' 8-byte reads spread over all banks
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    char *tile = reinterpret_cast<char *>(gm_lds + bt.K) + (size_t)wid * (GM_ROWS * PITCH);

    const int grp = blockIdx.x;
    const int mi = gv_find(bt.grp_begin, grp);
    const GemvMat &M = bt.mat[mi];
    const int row0 = (grp - bt.grp_begin[mi]) * ROWS;
    const int d_in = M.d_in, last_row = M.d_out - 1, m = bt.m;
    const int64_t row_bytes = M.row_bytes;
    const int n_chunks = d_in / GM_CHUNK;

    // The chunk's packed bytes of the workgroup's rows -- BITS 16-byte pieces per row -- are loaded with consecutive
    // lanes on consecutive pieces (piece 64 i + lane of the row-major ROWS x BITS array) and laid down in LDS row by row.
    // Rows past the end of the matrix re-read the last row (their results are not stored); lanes past the last piece
    // read and write that one once more.
    constexpr int PIECES = (ROWS * BITS + 63) / 64;
    auto piece_row = [&](int i) { return min(64 * i + lane, ROWS * BITS - 1) / BITS; };
    auto piece_col = [&](int i) { return 16 * (min(64 * i + lane, ROWS * BITS - 1) % BITS); };
    uint32_t src_off[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) src_off[i] = (uint32_t)min(row0 + piece_row(i), last_row) * (uint32_t)row_bytes + piece_col(i);
    const uint32_t z_lane = (uint32_t)(h * 16 * 256 + r * 8) * 2;     // bytes; padded rows exist and are zero

    gv_f32x16_t acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;

    // Wave w takes the chunks w, w + 8, ...: at any time the eight waves read neighbouring pieces of the same rows.
    //   Loads come back in the order they were asked for, so an instruction's activations (from L2) must not be asked for behind
    // the next chunk's packed bytes (from memory), or it waits for those.  Hence a ring of ZB instructions' activations, a slot
    // filled again as soon as its instruction has been issued, and the packed bytes of the wave's next chunk requested when all
    // activations of this one are on their way.  All loads are buffer loads without a branch around them, out of range where
    // there is no next chunk: behind a branch the compiler waits for what either side may have asked for.  The first chunk's are
    // requested before the codebook is staged.  (A wave without a chunk reads another's.)  The four launches of a 7B layer at 32
    // rows, in a trace: 24.2 + 10.2 + 20 + 17.4 us, so 21.6 + 7.8 + 18 + 15.0; 4096 x 11008, 64 rows, a call: 31.4 -> 26.0.
    //   Ring: four slots for one tile of activation rows, two for two, what the registers hold.
    gv_u32x4_t v[PIECES];
    const int packed_bytes = M.d_out * (int)row_bytes;
    auto load_packed = [&](int ch, bool wanted) {
        const int at = ch * (16 * BITS);
        const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(M.packed + at), 0, wanted ? packed_bytes - at : 0, 0x00020000);
#pragma unroll
        for (int i = 0; i < PIECES; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(res, src_off[i], 0, 0);
    };
    constexpr int ZB = MT == 1 ? 4 : 2;
    gv_u32x4_t zb[MT][ZB];
    // the activations of instruction `step` of chunk ch
    auto load_zb = [&](int ch, int step, bool wanted) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const char *at = reinterpret_cast<const char *>(M.Z) + ((int64_t)t * n_chunks + ch) * (32 * 512);
            const auto res = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(at), 0, wanted ? 32 * 512 : 0, 0x00020000);
            zb[t][step % ZB] = __builtin_amdgcn_raw_buffer_load_b128(res, z_lane + step * 512, 0, 0);
        }
    };
    const int first_ch = min(wid, n_chunks - 1);
    load_packed(first_ch, true);
#pragma unroll
    for (int j = 0; j < ZB; ++j) load_zb(first_ch, j, true);
    const int row = row0 + r;
    const float norm = M.norms[min(row, last_row)];
    {   // stage the codebook, rounded to bf16
        constexpr int KC = 1 << BITS, PER = (KC + GM_THREADS - 1) / GM_THREADS;
        const float2 *cbk = reinterpret_cast<const float2 *>(bt.codebook);
        float2 c[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) c[j] = cbk[min((int)threadIdx.x + j * GM_THREADS, KC - 1)];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const gv_f32x2_t u = {c[j].x, c[j].y};
            if (KC % GM_THREADS == 0 || (int)threadIdx.x + j * GM_THREADS < KC) cbh[threadIdx.x + j * GM_THREADS] = __builtin_bit_cast(uint32_t, __builtin_convertvector(u, gv_bf16x2_t));
        }
        __syncthreads();
    }
#pragma unroll 1
    for (int ch = wid; ch < n_chunks; ch += GM_WAVES) {
        const bool more = ch + GM_WAVES < n_chunks;
        const int next_ch = more ? ch + GM_WAVES : ch;
        // the chunk's packed bytes go through LDS: written piece by piece, read back as the lane's stream of 64 pairs
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            gv_u32x2_t *dst = reinterpret_cast<gv_u32x2_t *>(tile + piece_row(i) * PITCH + piece_col(i));
            dst[0] = gv_u32x2_t{v[i][0], v[i][1]};
            dst[1] = gv_u32x2_t{v[i][2], v[i][3]};
        }
        uint32_t w[2 * BITS];
        const gv_u32x2_t *src = reinterpret_cast<const gv_u32x2_t *>(tile + (r & (ROWS - 1)) * PITCH + 8 * BITS * h);
#pragma unroll
        for (int q = 0; q < BITS; ++q) {
            const gv_u32x2_t x2 = src[q];
            w[2 * q] = x2[0];
            w[2 * q + 1] = x2[1];
        }
        gv_u32x4_t a[2];                                        // an instruction's codewords are gathered while the one before it runs
        auto gather = [&](int step) {                           // pairs 4 step .. 4 step + 3 of the lane's 64
#pragma unroll
            for (int f = 0; f < 4; ++f)
                a[step & 1][f] = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(cbh) + gm_field_x4<BITS>(w, 4 * step + f));
        };
        gather(0);
#pragma unroll
        for (int step = 0; step < 16; ++step) {
            if (step + 1 < 16) gather(step + 1);
            const gv_bf16x8_t av = __builtin_bit_cast(gv_bf16x8_t, a[step & 1]);
#pragma unroll
            for (int t = 0; t < MT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(gv_bf16x8_t, zb[t][step % ZB]), acc[t], 0, 0, 0);
            if (step + ZB < 16) load_zb(ch, step + ZB, true);
            else load_zb(next_ch, step + ZB - 16, more);
            __builtin_amdgcn_sched_barrier(0);
            if (step + ZB == 15) {
                load_packed(next_ch, more);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // The eight waves' tiles, summed in wave order.  All waves leave theirs in LDS (over the packed tiles: everybody is done
    // with those), 32 activation rows at a time, then each takes an eighth of the sums, lanes along the weight rows: 128
    // consecutive bytes of Y per half-wave.  Wave 0 alone with lanes along the activation rows (112 reads and 16 stores of
    // 64 scattered words) took longer: the four calls of a 7B
    // layer at 32 activation rows 104 us, so 94.
    constexpr int RED_PITCH = GM_ROWS + 1;                      // floats of one activation row's 32 sums
    constexpr int RED_WAVE = 32 * RED_PITCH;
    const bool row_ok = r < ROWS && row <= last_row;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        __syncthreads();
        float *dst = red + wid * RED_WAVE + r * RED_PITCH + 4 * h;     // the accumulator's column is the activation row
#pragma unroll
        for (int i = 0; i < 16; ++i) dst[8 * (i >> 2) + (i & 3)] = acc[t][i];   // accumulator i of half h: the tile's row
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int col = 16 * q + 2 * wid + h, tok = 32 * t + col;
            const float *src = red + col * RED_PITCH + r;
            float s = src[0];
#pragma unroll
            for (int w2 = 1; w2 < GM_WAVES; ++w2) s += src[w2 * RED_WAVE];
            if (row_ok && tok < m) M.Y[(int64_t)tok * M.ldy + row] = norm * s;
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// More than 64 activation rows: the same product in tiles of 128 weight rows x 128 TT activation rows, 8 waves (2 x 4) of
// 64 x 32 TT each.
//   A stage is 4 matrix instructions of depth (64 of the 256 columns of a chunk).  The weights' side of a stage is unpacked
// once per workgroup: a lane takes 8 pairs of one (row, half), gathers their bf16 codewords and leaves them in LDS in the
// order the A operand is read; the activations go from memory straight into LDS (k_rotate_tile wrote them in B's order).
// While stage s is multiplied the weights of stage s + 1 are unpacked (two buffers) and the activations of the stages after it
// are under way (three to five: an L2 round trip is longer than a stage).
//   One barrier per stage, before its last quarter: by then a wave has read all operands of the stage and left its part of the
// next one's, and the products still to come hide the first reads of the next stage.  LDS accesses and requests are dealt out
// between the products, two or three to each: in a block before them they and the products waited for each other, two waves
// per SIMD in step.  The activations are requested with buffer instructions: the compiler counts those and waits for a piece of
// weights alone, where it waited for all that was under way, once a chunk, with flat ones.  8192 x 4096, 1024 rows, 256 tiles of
// 128 x 256: 99 -> 88 us a call, of which 9 for the rotation.
//   What bounds it: the LDS, with 128 KB of operand reads, 4 K codeword gathers and 48 KB of writes per stage of 2000 cycles
// (210 instructions, two thirds of the time with the writes from memory), and the matrix cores, busy half the time (without
// the products 80 us; without gathers, unpacked weights and requests 72).  An unpacked operand has to serve many activation
// rows; the kernel for up to 64 rows unpacks the matrix again for every launch.
//   Summation order: exactly that of k_qgemm -- the chunks w, w + 8, ... summed in an accumulator of their own for
// w = 0 .. 7, those eight then added in order -- so a row of Y has the same bits whatever m is and whichever of the two
// kernels computes it; that is why the kernel keeps two accumulators.
constexpr int GW_ROWS = 128;               // weight rows of a workgroup
constexpr int GW_WAVES = 8, GW_THREADS = GW_WAVES * WAVE;
constexpr int GW_CUS = 256;                // one workgroup per CU at a time
constexpr int GW_STAGE = 4;                // matrix instructions of depth per stage

constexpr int gw_buffers(int tt) { return tt == 2 ? 3 : 5; }    // stages of activations in LDS: 136 and 120 KB in all

template <int BITS, int TT> __device__ __forceinline__ void gw_tile(const GemvBatch &bt, const GemvMat &M, int local) {
    constexpr int BUFS = gw_buffers(TT);
    constexpr int TILES = 4 * TT;                               // 32-row tiles of activation rows
    constexpr int KC = 1 << BITS;
    constexpr uint32_t A_BYTES = 4 * GW_STAGE * 1024, Z_BYTES = TILES * GW_STAGE * 1024;
    constexpr uint32_t A_AT = KC * 4;                           // after the K codewords, (bf16 c0) | (bf16 c1) << 16:
                                                                // 2 buffers [4 tiles of 32 rows][4 instructions][64 lanes] x 16 bytes
    constexpr uint32_t Z_AT = A_AT + 2 * A_BYTES;               // BUFS buffers [TILES][2 halves][4 instructions][32 rows] x 16 bytes
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int wn = wid & 1, wm = wid >> 1;

    const int m = bt.m, d_out = M.d_out, last_row = d_out - 1;
    const int tok_tiles = (m + 31) >> 5, m_tiles = (tok_tiles + TILES - 1) / TILES;
    // Workgroup b runs on XCD b mod 8: the activation tiles of one weight tile follow one another on the same XCD, so the
    // packed rows come from its L2 after the first.
    const int n_tiles = (d_out + GW_ROWS - 1) / GW_ROWS;
    int nt, mt;
    {
        const int whole = n_tiles / 8 * 8 * m_tiles;            // the last n_tiles mod 8 weight tiles in plain order
        if (local < whole) {
            const int x = local & 7, q = local >> 3;
            nt = x + 8 * (q / m_tiles);
            mt = q - q / m_tiles * m_tiles;
        } else {
            const int q = local - whole;
            nt = n_tiles / 8 * 8 + q / m_tiles;
            mt = q - q / m_tiles * m_tiles;
        }
    }
    const int row0 = nt * GW_ROWS, tile0 = mt * TILES;
    const int n_chunks = M.d_in / GM_CHUNK;

    {   // stage the codebook, rounded to bf16
        const float2 *cbk = reinterpret_cast<const float2 *>(bt.codebook);
        for (int i = threadIdx.x; i < KC; i += GW_THREADS) {
            const float2 c = cbk[i];
            const gv_f32x2_t v = {c.x, c.y};
            lds_write<uint32_t>(4 * i, __builtin_bit_cast(uint32_t, __builtin_convertvector(v, gv_bf16x2_t)));
        }
    }

    // Stage q of a chunk: waves w and w + 4 unpack the w-th 32 rows; this wave's part is 8 pairs, BITS bytes from byte
    // (2 q + part) BITS of the lane's half of the row.  A lane holds the dwords that cover them (moved back where they would
    // reach past the half, i.e. possibly past the matrix), four stages ahead.
    constexpr int PIECE = (BITS + 3) / 4 + (BITS % 4 ? (BITS % 4 > 1 ? 1 : 0) : 0);
    static_assert(PIECE == (BITS == 11 ? 4 : BITS == 7 ? 3 : 2), "dwords that cover a piece at any byte offset");
    const int part = wid >> 2;
    const uint8_t *src_row = M.packed + (int64_t)min(row0 + 32 * (wid & 3) + r, last_row) * M.row_bytes + h * (8 * BITS);
    uint32_t pc[4][PIECE];
    auto load_piece = [&](int ch, int q, uint32_t (&w)[PIECE]) {
        typedef uint32_t u32xp_t __attribute__((ext_vector_type(PIECE)));
        typedef u32xp_t u32xp_a4_t __attribute__((aligned(4)));
        const int at = min(((2 * q + part) * BITS) & ~3, 8 * BITS - 4 * PIECE);
        const u32xp_t v = *reinterpret_cast<const u32xp_a4_t *>(src_row + (int64_t)ch * (16 * BITS) + at);
#pragma unroll
        for (int i = 0; i < PIECE; ++i) w[i] = v[i];
    };
    // the piece's 8 fields from bit 0 on
    auto align_piece = [&](const uint32_t (&w)[PIECE], int q, uint32_t (&f)[3]) {
        const bool back = q == 3 && part == 1 && BITS != 8;     // the one piece whose dwords were moved back, by 4 bytes
        const uint32_t sh = (((2 * q + part) * BITS) & 3) * 8;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            auto dw = [&](int k) { return k < PIECE ? w[k] : 0u; };
            const uint32_t lo = back ? dw(i + 1) : dw(i), hi = back ? dw(i + 2) : dw(i + 1);
            f[i] = BITS == 8 ? lo : __builtin_amdgcn_alignbit(hi, lo, sh);
        }
    };
    // activations of stage q of a chunk: 1 KB pieces (two instructions of one half of one tile), 2 TT per wave
    const int my_tile = wid * TT / 2;
    const char *zsrc = reinterpret_cast<const char *>(M.Z) + (int64_t)min(tile0 + my_tile, tok_tiles - 1) * n_chunks * 16384 +
                       (TT == 1 ? (wid & 1) * 8192 : 0);        // tiles past the end repeat the last (not stored)
    const auto zres = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(zsrc), 0, n_chunks * 16384 - (TT == 1 ? (wid & 1) * 8192 : 0), 0x00020000);
    auto request_z = [&](int ch, int q, int u, uint32_t buf) {     // the u-th of them; buf: byte offset of the buffer
            __builtin_amdgcn_raw_ptr_buffer_load_lds(zres, reinterpret_cast<__attribute__((address_space(3))) void *>(Z_AT + buf + (wid * 2 * TT + u) * 1024u), 16,
                                                     lane * 16, ch * 16384 + (u >> 1) * 8192 + q * 2048 + (u & 1) * 1024, 0, 0);
    };
    const uint32_t a_write = A_AT + (uint32_t)((wid & 3) * GW_STAGE + 2 * part) * 1024 + lane * 16;
    const uint32_t a_read = A_AT + (uint32_t)(2 * wn) * (GW_STAGE * 1024) + lane * 16;
    const uint32_t z_read = Z_AT + (uint32_t)(wm * TT) * 4096 + h * 2048 + r * 16;
    // the i-th codeword of a piece
    auto gather = [&](const uint32_t (&f)[3], int i) {
        const int bit = i * BITS, word = bit >> 5, off = bit & 31;
        const uint32_t v = (off + BITS <= 32) ? (f[word] >> off) : __builtin_amdgcn_alignbit(f[word + 1], f[word], off);
        return lds_read<uint32_t>((v & (KC - 1u)) << 2);
    };

    gv_f32x16_t acc[2][TT], total[2][TT];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][t][i] = total[a][t][i] = 0.0f;
    // operands of a stage's instructions, a set of registers each
    gv_bf16x8_t av[GW_STAGE][2], bv[GW_STAGE][TT];
    constexpr int READS = 2 + TT, PRODUCTS = 2 * TT;            // of one instruction's depth
    auto operand = [&](int j, int i, uint32_t a_buf, uint32_t z_buf) {   // the i-th read, in the order of their use
        if (i == 0 || i == READS - 1) {
            const int a = i == 0 ? 0 : 1;
            av[j][a] = lds_read<gv_bf16x8_t>(a_read + a_buf + (a * GW_STAGE + j) * 1024);
        } else {
            bv[j][i - 1] = lds_read<gv_bf16x8_t>(z_read + z_buf + (i - 1) * 4096 + j * 512);
        }
    };
    auto product = [&](int i) {                                 // the i-th of a stage
        const int j = i / PRODUCTS, a = i % PRODUCTS / TT, t = i % TT;
        acc[a][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[j][a], bv[j][t], acc[a][t], 0, 0, 0);
    };

#pragma unroll
    for (int q = 0; q < 4; ++q) load_piece(0, q, pc[q]);
    // the chunk after c of segment s: the next of the segment (+ 8) or the first of the next segment; at the end the same again (unused)
    auto after = [&](int c, int s, int &c2, int &s2) {
        c2 = c + GM_WAVES;
        s2 = s;
        if (c2 >= n_chunks) c2 = s2 = s + 1;
        if (s2 >= GM_WAVES || c2 >= n_chunks) {
            c2 = c;
            s2 = s;
        }
    };
    int ch = 0, seg = 0, next, next_seg, later, later_seg;
    after(ch, seg, next, next_seg);
#pragma unroll
    for (int q = 0; q < BUFS; ++q)
#pragma unroll
        for (int u = 0; u < 2 * TT; ++u) request_z(q < 4 ? 0 : next, q & 3, u, q * Z_BYTES);
    __syncthreads();                                            // the codebook is staged
    {
        uint32_t f[3];
        align_piece(pc[0], 0, f);
#pragma unroll
        for (int i = 0; i < 2; ++i) lds_write(a_write + 1024 * i, gv_u32x4_t{gather(f, 4 * i), gather(f, 4 * i + 1), gather(f, 4 * i + 2), gather(f, 4 * i + 3)});
        load_piece(next, 0, pc[0]);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt(0): the wave's activations have landed
    __syncthreads();
#pragma unroll
    for (int i = 0; i < READS; ++i) operand(0, i, 0, 0);
    uint32_t z_now = 0;                                         // the buffer of this stage's activations
#pragma unroll 1
    for (int left = n_chunks; left > 0; --left) {
        after(next, next_seg, later, later_seg);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cur = q & 1, nxt = cur ^ 1;
            const uint32_t z_next = z_now == (BUFS - 1) * Z_BYTES ? 0 : z_now + Z_BYTES;
            // What the wave has to ask of LDS and memory, a little before each product, so that both go on at once: first the
            // rest of this stage's operands and the weights of the next stage, ...
            uint32_t f[3];
            align_piece(pc[(q + 1) & 3], (q + 1) & 3, f);
            gv_u32x4_t cw[2];
            constexpr int TASKS = 3 * READS + 8 + 3, BEFORE = 3 * PRODUCTS;
            auto task = [&](int n) {
                if (n < READS) return operand(1, n, cur * A_BYTES, z_now);
                n -= READS;
                if (n < 4) return (void)(cw[0][n] = gather(f, n));
                n -= 4;
                if (n < READS) return operand(2, n, cur * A_BYTES, z_now);
                n -= READS;
                if (n < 4) return (void)(cw[1][n] = gather(f, 4 + n));
                n -= 4;
                if (n < 1) return lds_write(a_write + nxt * A_BYTES, cw[0]);
                n -= 1;
                if (n < READS) return operand(3, n, cur * A_BYTES, z_now);
                n -= READS;
                if (n < 1) return load_piece(q == 3 ? later : next, (q + 1) & 3, pc[(q + 1) & 3]);   // in the place of the used one
                lds_write(a_write + nxt * A_BYTES + 1024, cw[1]);
            };
#pragma unroll
            for (int i = 0; i < BEFORE; ++i) {
#pragma unroll
                for (int n = 0; n < TASKS; ++n)
                    if (n * (BEFORE - 1) / TASKS == i) task(n);
                product(i);
                __builtin_amdgcn_sched_barrier(0);
            }
            // Of this stage's buffers all that the wave needs is in its registers, its part of the next stage's weights is written,
            // and its next activations have landed: since their request a piece, then BUFS - 2 times the 2 TT loads of a stage and a piece.
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(BUFS - 1 + (BUFS - 2) * 2 * TT) : "memory");
            __builtin_amdgcn_sched_barrier(0);
            // ... then the next stage's first operands and, into this stage's buffer, the activations BUFS stages ahead.
#pragma unroll
            for (int i = BEFORE; i < 4 * PRODUCTS; ++i) {
#pragma unroll
                for (int n = 0; n < READS; ++n)
                    if (n * PRODUCTS / READS == i - BEFORE) operand(0, n, nxt * A_BYTES, z_next);
                request_z(q + BUFS < 4 ? ch : q + BUFS < 8 ? next : later, (q + BUFS) & 3, i - BEFORE, z_now);
                product(i);
                __builtin_amdgcn_sched_barrier(0);
            }
            z_now = z_next;
        }
        if (left == 1 || next_seg != seg) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int t = 0; t < TT; ++t) {
                    total[a][t] = seg == 0 ? acc[a][t] : total[a][t] + acc[a][t];
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[a][t][i] = 0.0f;
                }
        }
        ch = next;
        seg = next_seg;
        next = later;
        next_seg = later_seg;
    }

    // The norms first, all of them, then four consecutive weight rows per store: a load between two stores would wait for
    // the first to reach memory.
    float nr[2][16];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 16; ++i) nr[a][i] = M.norms[min(row0 + 32 * (2 * wn + a) + 8 * (i >> 2) + 4 * h + (i & 3), last_row)];
    typedef gv_f32x4_t f32x4_a4_t __attribute__((aligned(4)));
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            const int tok = 32 * (tile0 + wm * TT + t) + r;     // the accumulator's column is the activation row
            if (tok >= m) continue;
            float *dst = M.Y + (int64_t)tok * M.ldy;
#pragma unroll
            for (int g = 0; g < 4; ++g) {                       // accumulators 4 g .. 4 g + 3 of half h
                const int row = row0 + 32 * (2 * wn + a) + 8 * g + 4 * h;
                gv_f32x4_t y;
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i] = nr[a][4 * g + i] * total[a][t][4 * g + i];
                if (row + 3 <= last_row) {
                    *reinterpret_cast<f32x4_a4_t *>(dst + row) = y;
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (row + i <= last_row) dst[row + i] = y[i];
                }
            }
        }
    }
}

template <int BITS>
__global__ __launch_bounds__(GW_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_qgemm_wide(GemvBatch bt) {
    const int mi = gv_find(bt.grp_begin, blockIdx.x);
    const GemvMat &M = bt.mat[mi];
    const int local = (int)blockIdx.x - bt.grp_begin[mi];
    if (M.tok_tiles == 2) gw_tile<BITS, 2>(bt, M, local);
    else gw_tile<BITS, 1>(bt, M, local);
}

bool matmul_supported(const Problem &p, int m) {
    const int unit = p.block > 16 ? p.block : 16;
    if (p.d_in % unit || p.block < 64) return false;
    if (p.bits != 7 && p.bits != 8 && p.bits != 11) return false;
    if (m > GV_MAX_M) return p.d_in % GM_CHUNK == 0;               // the matrix-core kernels walk 256-column chunks
    return m >= 1;
}

// Whether m activation rows are better taken whole, by the wide kernel, than 64 at a time.  A wide workgroup walks all columns,
// 0.6 us per 64 of them, whatever the number of rows; the smaller kernel unpacks the matrix once per 64 rows, but spreads a row over
// its waves.  So up to two tiles of 64 the smaller one is sooner done; with three where the rows are longer than WIDE_SHORT and the
// wide tiles leave most of the chip idle, or fill a last round badly; with four where they are long and leave most of it idle.
//   In us, tiles / wide, at 11 bits (7 and 8 alike).  129 rows: 256 x 2048 33.6 / 32.1, 4096 x 1024 31.5 / 22.2, 2048 x 2560 38.3 /
// 36.3, 5120 x 5120 63.0 / 59.9, 8192 x 4096 60.5 / 51.9; but 2048 x 3072 39.1 / 41.3, 4096 x 4096 42.8 / 50.2, 4096 x 11008 80.8 /
// 114, 11008 x 4096 twice (344 tiles of 128 x 128) 91.2 / 94.6.  256 rows: 4096 x 4096 57.1 / 51.8, 1024 x 5120 62.8 / 61.2, 5120 x
// 13824 184 / 138; but 2048 x 5632 64.0 / 66.5, 4096 x 11008 107 / 114, 1024 x 14336 113 / 146.  128 rows: 4096 x 1024 21.9 / 22.2, others
// 25 % to three times.  257 rows: 1024 x 14336 140 / 147, others wide.
bool matmul_wide(const MatmulItem *items, int n, int m) {
    constexpr int WIDE_SHORT = 2560, WIDE_LONG = 5120;
    if (m <= 2 * GM_MAX_M) return false;
    int64_t groups = 0;                                         // of 128 x 128, one round of them on the chip
    int longest = 0;
    for (int i = 0; i < n; ++i) {
        if (items[i].d_in >= 1 << 25) return false;             // a tile's activations: 64 bytes a column, 32-bit offsets
        groups += (int64_t)((items[i].d_out + GW_ROWS - 1) / GW_ROWS) * ((m + 127) / 128);
        longest = std::max(longest, items[i].d_in);
    }
    if (m > 4 * GM_MAX_M) return true;
    if (m > 3 * GM_MAX_M) return longest <= WIDE_LONG || 4 * groups > GW_CUS;
    const int64_t rounds = (groups + GW_CUS - 1) / GW_CUS;
    return longest <= WIDE_SHORT || (16 * groups >= 5 * GW_CUS && (rounds == 1 || 4 * groups >= 3 * GW_CUS * rounds));
}

size_t matmul_workspace_bytes(int d_in, int d_out, int m) {
    (void)d_out;
    // the rotated activations: fp32 rows, or (matrix-core kernel) bf16 rows padded to a multiple of 32 rows
    const size_t bytes = m <= GV_MAX_M ? (size_t)m * d_in * sizeof(float) : (size_t)((m + 31) / 32 * 32) * d_in * sizeof(uint16_t);
    return (bytes + 15) / 16 * 16;
}

template <int XDTYPE>
static hipError_t launch_rotate(const GemvBatch &bt, int block, hipStream_t stream) {
    const unsigned blocks = (unsigned)((bt.rot_begin[bt.n] + GV_WAVES - 1) / GV_WAVES);
#define QAMW_ROT(BB) \
    case BB: hipLaunchKernelGGL((k_rotate_x<XDTYPE, BB>), dim3(blocks), dim3(GV_THREADS), 0, stream, bt); break;
    switch (block) {
        QAMW_ROT(64) QAMW_ROT(128) QAMW_ROT(256) QAMW_ROT(512) QAMW_ROT(1024)
        default: return hipErrorNotSupported;
    }
#undef QAMW_ROT
    return hipGetLastError();
}
// rows: activation rows per workgroup, 8 or 16
template <int XDTYPE>
static hipError_t launch_rotate_tile(const GemvBatch &bt, int rows, int block, hipStream_t stream) {
    const unsigned blocks = (unsigned)bt.rot_begin[bt.n];
#define QAMW_ROT(BB) \
    case BB: \
        if (rows == 16) hipLaunchKernelGGL((k_rotate_tile<XDTYPE, BB, 2, true>), dim3(blocks), dim3(GM_THREADS), 0, stream, bt); \
        else if (bt.m > GM_MAX_M) hipLaunchKernelGGL((k_rotate_tile<XDTYPE, BB, 1, true>), dim3(blocks), dim3(GM_THREADS), 0, stream, bt); \
        else hipLaunchKernelGGL((k_rotate_tile<XDTYPE, BB, 1, false>), dim3(blocks), dim3(GM_THREADS), 0, stream, bt); \
        break;
    switch (block) {
        QAMW_ROT(64) QAMW_ROT(128) QAMW_ROT(256) QAMW_ROT(512) QAMW_ROT(1024)
        default: return hipErrorNotSupported;
    }
#undef QAMW_ROT
    return hipGetLastError();
}

template <int BITS, int RB>
static hipError_t launch_qgemv_rb(const GemvBatch &bt, hipStream_t stream) {
    const unsigned blocks = (unsigned)bt.grp_begin[bt.n];
#define QAMW_GV(MM, AH) hipLaunchKernelGGL((k_qgemv<BITS, MM, RB, AH>), dim3(blocks), dim3(GV_THREADS), 0, stream, bt)
    if constexpr (RB > 0) {                                     // the self-rotating kernels exist for one and two rows
        bool one_step = true;                                   // in every wave
        for (int i = 0; i < bt.n; ++i) one_step = one_step && bt.mat[i].n_slabs * (bt.mat[i].rows_per_wg / GV_RG) <= GV_WAVES;
        if (bt.m == 1 && one_step) QAMW_GV(1, 1);
        else if (bt.m == 1) QAMW_GV(1, 2);
        else if (bt.m == 2 && blocks <= GV_AHEAD_MAX_WGS_2) QAMW_GV(2, 2);
        else if (bt.m == 2) QAMW_GV(2, 0);
        else return hipErrorNotSupported;
    } else {
        if (bt.m == 1) QAMW_GV(1, 0);
        else if (bt.m == 2) QAMW_GV(2, 0);
        else if (bt.m <= 4) QAMW_GV(4, 0);
        else QAMW_GV(8, 0);
    }
#undef QAMW_GV
    return hipGetLastError();
}
// rotate_block: 0, or the block size when the product kernel is to rotate the activations itself
template <int BITS>
static hipError_t launch_qgemv(const GemvBatch &bt, int rotate_block, hipStream_t stream) {
    switch (rotate_block) {
        case 0: return launch_qgemv_rb<BITS, 0>(bt, stream);
        case 64: return launch_qgemv_rb<BITS, 64>(bt, stream);
        case 128: return launch_qgemv_rb<BITS, 128>(bt, stream);
        case 256: return launch_qgemv_rb<BITS, 256>(bt, stream);
        case 512: return launch_qgemv_rb<BITS, 512>(bt, stream);
        case 1024: return launch_qgemv_rb<BITS, 1024>(bt, stream);
        default: return hipErrorNotSupported;
    }
}

template <int BITS>
static hipError_t launch_qgemm(const GemvBatch &bt, hipStream_t stream) {
    const unsigned blocks = (unsigned)bt.grp_begin[bt.n];
    const int mt = (bt.m + 31) / 32;
    const size_t red_bytes = (size_t)GM_WAVES * 32 * (GM_ROWS + 1) * sizeof(float);
    const size_t tile_bytes = (size_t)GM_WAVES * GM_ROWS * (16 * BITS + 8);
    const size_t lds = (size_t)bt.K * sizeof(uint32_t) + (red_bytes > tile_bytes ? red_bytes : tile_bytes);
#define QAMW_GM(MM, RR) hipLaunchKernelGGL((k_qgemm<BITS, MM, RR>), dim3(blocks), dim3(GM_THREADS), lds, stream, bt)
    if (mt == 1 && bt.gm_rows == GM_ROWS) QAMW_GM(1, GM_ROWS);
    else if (mt == 1) QAMW_GM(1, GM_ROWS / 2);
    else if (bt.gm_rows == GM_ROWS) QAMW_GM(2, GM_ROWS);
    else QAMW_GM(2, GM_ROWS / 2);
#undef QAMW_GM
    return hipGetLastError();
}

template <int BITS>
static hipError_t launch_qgemm_wide(const GemvBatch &bt, hipStream_t stream) {
    auto bytes = [](int tt) { return ((size_t)4 << BITS) + (size_t)(2 * 4 + gw_buffers(tt) * 4 * tt) * GW_STAGE * 1024; };
    const size_t lds = std::max(bytes(1), bytes(2));            // more than the 64 KB that a workgroup has without asking
    static std::atomic<uint64_t> done{0};                       // the devices on which it was asked for
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorNotSupported;
    if (!(done.load(std::memory_order_acquire) & (1ull << dev))) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_qgemm_wide<BITS>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        done.fetch_or(1ull << dev, std::memory_order_release);
    }
    hipLaunchKernelGGL((k_qgemm_wide<BITS>), dim3((unsigned)bt.grp_begin[bt.n]), dim3(GW_THREADS), lds, stream, bt);
    return hipGetLastError();
}

// Y_i = X_i W_i^T for n <= QAMW_MATMUL_MAX_BATCH matrices that share codebook, bits, block, m and the element type
// of X.  workspace: the sum of matmul_workspace_bytes() over the items, 16-byte aligned.
// Returns hipErrorNotSupported (nothing launched) outside the supported shapes.  variant: 0, or 1 / 2 to force the
// two-launch / the self-rotating form of the vector kernel.
hipError_t launch_matmul_batch(const MatmulItem *items, int n, int xdtype, int m, const Problem &p, void *workspace, int variant) {
    if (n < 1 || n > QAMW_MATMUL_MAX_BATCH || p.K != (1 << p.bits)) return hipErrorNotSupported;   // the kernels size the codebook from the bit width
    // The vector kernel's offsets into a group of rows are 32 bits: rows of 2^28 bytes and more one at a time.
    constexpr int64_t LONG_ROW = (int64_t)1 << 28;
    for (int i = 0; i < n && m <= GV_MAX_M; ++i) {
        const int64_t row_bytes = (((int64_t)(items[i].d_in / 2) * p.bits + 31) / 32) * 4;
        if (row_bytes < LONG_ROW || items[i].d_out == 1) continue;
        for (int k = 0; k < n; ++k) {
            const int64_t kb = (((int64_t)(items[k].d_in / 2) * p.bits + 31) / 32) * 4;
            const int rows = kb < LONG_ROW ? items[k].d_out : 1;
            for (int row = 0; row < items[k].d_out; row += rows) {
                MatmulItem one = items[k];
                one.d_out = rows;
                one.packed += row * kb;
                one.norms += row;
                one.Y += row;
                const hipError_t e = launch_matmul_batch(&one, 1, xdtype, m, p, workspace, variant);
                if (e != hipSuccess) return e;
            }
        }
        return hipSuccess;
    }
    GemvBatch bt;
    int64_t rot = 0, groups = 0;
    char *ws = static_cast<char *>(workspace);
    // Matrix-core kernel: the products with the longest rows go first in the grid.  Their workgroups take longest (one
    // workgroup walks whole rows); started last, they would run on alone after everything else has finished.  The
    // order inside a launch changes no result.
    int order[QAMW_MATMUL_MAX_BATCH];
    for (int i = 0; i < n; ++i) order[i] = i;
    if (m > GV_MAX_M)
        std::stable_sort(order, order + n, [&](int a, int b) { return items[a].d_in > items[b].d_in; });
    // Matrix-core kernel: a launch whose matrices make at most GM_HALF_TILE_MAX_WGS workgroups of 32 rows (one 4096-row
    // projection makes 128) is cut into workgroups of 16 rows, so that it reaches every CU; a row's result does not
    // depend on the cut.
    int64_t tiles32 = 0;
    for (int i = 0; i < n; ++i) tiles32 += (items[i].d_out + GM_ROWS - 1) / GM_ROWS;
    bt.gm_rows = tiles32 <= GM_HALF_TILE_MAX_WGS ? GM_ROWS / 2 : GM_ROWS;
    // More than 64 activation rows: tiles of 256 of them where those make enough workgroups for the chip, else of 128.
    const bool wide = m > GM_MAX_M;
    auto wide_groups = [&](const MatmulItem &it, int tt) {
        return (int64_t)((it.d_out + GW_ROWS - 1) / GW_ROWS) * ((m + 128 * tt - 1) / (128 * tt));
    };
    int64_t groups256 = 0;
    for (int i = 0; i < n; ++i) groups256 += wide_groups(items[i], 2);
    const int tt = groups256 >= GW_CUS ? 2 : 1;
    // Matrix-core kernels: 16 activation rows per workgroup of the rotation where those are at least one for every CU.
    int64_t slabs = 0;
    for (int i = 0; i < n; ++i) slabs += (items[i].d_in + GV_SLAB - 1) / GV_SLAB;
    const int rot_rows = (m + 31) / 32 * 2 * slabs >= GW_CUS ? 16 : 8;
    for (int i = 0; i < n; ++i) {
        const MatmulItem &it = items[order[i]];
        Problem q = p;
        q.d_in = it.d_in;
        q.d_out = it.d_out;
        if (!matmul_supported(q, m) || (reinterpret_cast<uintptr_t>(it.packed) & 3)) return hipErrorNotSupported;
        GemvMat &M = bt.mat[i];
        M.X = it.X;
        M.packed = it.packed;
        M.norms = it.norms;
        M.chan_scale = it.chan_scale;
        M.pair_sigma = it.pair_sigma;
        M.signs = it.signs;
        M.Y = it.Y;
        M.ldx = it.ldx;
        M.ldy = it.ldy;
        M.d_out = it.d_out;
        M.d_in = it.d_in;
        M.n_slabs = (M.d_in + GV_SLAB - 1) / GV_SLAB;
        M.sigma_default = (float)(1.0 / std::sqrt((double)M.d_in));
        M.row_bytes = (((int64_t)(M.d_in / 2) * p.bits + 31) / 32) * 4;
        M.Z = reinterpret_cast<float *>(ws);
        ws += matmul_workspace_bytes(M.d_in, M.d_out, m);
        // Rows per workgroup, from the matrix's own shape only (so a product gives the same bits alone and in a
        // batch): about GV_STEPS_PER_WG (slab, row group) steps per workgroup, halved while the matrix would
        // otherwise make fewer than GV_MIN_WGS workgroups.
        int groups_per_wg = GV_STEPS_PER_WG / M.n_slabs;
        if (groups_per_wg < 1) groups_per_wg = 1;
        if (groups_per_wg > GV_MAX_ROWS_PER_WG / GV_RG) groups_per_wg = GV_MAX_ROWS_PER_WG / GV_RG;
        while (groups_per_wg > 1 && (M.d_out + groups_per_wg * GV_RG - 1) / (groups_per_wg * GV_RG) < GV_MIN_WGS) groups_per_wg >>= 1;
        M.rows_per_wg = groups_per_wg * GV_RG;
        if (m > GV_MAX_M) {                                     // matrix-core kernel: one tile, or half of one, per workgroup
            if ((int64_t)M.d_out * M.row_bytes > 0x7fffffff) return hipErrorNotSupported;   // 32-bit byte offsets into the packed matrix
            M.rows_per_wg = bt.gm_rows;
        }
        bt.rot_begin[i] = (int)rot;
        bt.grp_begin[i] = (int)groups;
        M.tok_tiles = tt;
        rot += (int64_t)(m > GV_MAX_M ? (m + 31) / 32 * 32 / rot_rows : m) * M.n_slabs;
        groups += wide ? wide_groups(it, tt) : (M.d_out + M.rows_per_wg - 1) / M.rows_per_wg;
        if (groups > 0x3fffffff || rot > 0x3fffffff) return hipErrorNotSupported;
    }
    for (int i = n; i <= QAMW_MATMUL_MAX_BATCH; ++i) {
        bt.rot_begin[i] = (int)rot;
        bt.grp_begin[i] = (int)groups;
    }
    for (int i = n; i < QAMW_MATMUL_MAX_BATCH; ++i) bt.mat[i] = bt.mat[0];
    bt.n = n;
    bt.m = m;
    bt.K = p.K;
    bt.inv_sqrt_block = p.inv_sqrt_block;
    bt.codebook = p.codebook;
    bt.xdtype = xdtype;
    // One or two activation rows in a small launch (a forward pass issues one product, or the few that share an input,
    // per call): the product kernel rotates the activations itself.  Same results, one launch less.
    // (variant 1: never, 2: whenever there are one or two rows -- for tests and measurements)
    const bool self_rotate = m <= 2 && variant != 1 && (variant == 2 || groups <= GV_SELF_ROTATE_MAX_WGS);
    hipError_t e = hipSuccess;
    if (m > GV_MAX_M)
        e = xdtype == 0 ? launch_rotate_tile<0>(bt, rot_rows, p.block, p.stream) : launch_rotate_tile<1>(bt, rot_rows, p.block, p.stream);
    else if (!self_rotate)
        e = xdtype == 0 ? launch_rotate<0>(bt, p.block, p.stream) : launch_rotate<1>(bt, p.block, p.stream);
    if (e != hipSuccess) return e;
    if (wide) {
        // One product whose 256-row tiles leave most of the chip idle in the last round: the weight rows of that round go
        // into 128-row tiles, if those are at most a round, of the same launch (11008 x 4096, 1000 rows, 344 tiles: in a launch of
        // their own 136 us a call, so 132).
        const int m_tiles = (m + 255) / 256, n_tiles = (items[0].d_out + GW_ROWS - 1) / GW_ROWS;
        const int first = (int)(groups256 / GW_CUS * GW_CUS) / m_tiles, rest = (n_tiles - first) * ((m + 127) / 128);
        if (n == 1 && tt == 2 && first < n_tiles && rest <= GW_CUS) {
            GemvMat &M = bt.mat[0], &M2 = bt.mat[1];            // as two matrices
            M2 = M;
            M.d_out = first * GW_ROWS;
            M2.d_out -= M.d_out;
            M2.packed += (int64_t)M.d_out * M.row_bytes;
            M2.norms += M.d_out;
            M2.Y += M.d_out;
            M2.tok_tiles = 1;
            bt.n = 2;
            bt.grp_begin[1] = first * m_tiles;
            for (int i = 2; i <= QAMW_MATMUL_MAX_BATCH; ++i) bt.grp_begin[i] = first * m_tiles + rest;
        }
        if (p.bits == 11) return launch_qgemm_wide<11>(bt, p.stream);
        if (p.bits == 8) return launch_qgemm_wide<8>(bt, p.stream);
        return launch_qgemm_wide<7>(bt, p.stream);
    }
    if (m > GV_MAX_M) {
        if (p.bits == 11) return launch_qgemm<11>(bt, p.stream);
        if (p.bits == 8) return launch_qgemm<8>(bt, p.stream);
        return launch_qgemm<7>(bt, p.stream);
    }
    const int rb = self_rotate ? p.block : 0;
    if (p.bits == 11) e = launch_qgemv<11>(bt, rb, p.stream);
    else if (p.bits == 8) e = launch_qgemv<8>(bt, rb, p.stream);
    else e = launch_qgemv<7>(bt, rb, p.stream);
    return e;
}

}  // namespace qamw
