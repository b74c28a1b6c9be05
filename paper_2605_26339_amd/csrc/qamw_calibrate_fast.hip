// Vectorised row norms and the shape-specialised pair-scale calibration (Eq. 1).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "qamw_front.hpp"

namespace qamw {

constexpr int CF_THREADS = 256;
constexpr int CF_WAVES = CF_THREADS / WAVE;
constexpr int CSLAB = 1024;
constexpr int CAL_ROWS = 8;     // calibration rows of a workgroup, one partial sum per pair
constexpr int CAL_THREADS = 512;
constexpr int CAL_WAVES = CAL_THREADS / WAVE;

// ---------------------------------------------------------------------------------------------
// Row norms, one wave per row.
// ---------------------------------------------------------------------------------------------
template <int DTYPE>
__global__ __launch_bounds__(CF_THREADS) void k_row_norms_vec(const void *__restrict__ W, int64_t ldw, int n_rows, int d_in,
                                                             const float *__restrict__ s, float *__restrict__ norms) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int row = __builtin_amdgcn_readfirstlane(blockIdx.x * CF_WAVES + (threadIdx.x >> 6));
    if (row >= n_rows) return;
    double s2[1];
    wave_rows_sum_of_squares<DTYPE, 1>(s2, W, row, 1, ldw, d_in, s, lane);
    if (lane == 0) norms[row] = (float)sqrt(s2[0]);
}

bool launch_row_norms_fast(const void *W, int dtype, int64_t ldw, int n_rows, const Problem &p, float *norms,
                           hipError_t *err) {
    const int v = dtype == 0 ? 4 : 8;
    if (p.d_in % v || ldw % v || (reinterpret_cast<uintptr_t>(W) & 15) || (reinterpret_cast<uintptr_t>(p.chan_scale) & 15))
        return false;
    dim3 grid((n_rows + CF_WAVES - 1) / CF_WAVES);
    if (dtype == 0)
        hipLaunchKernelGGL(k_row_norms_vec<0>, grid, dim3(CF_THREADS), 0, p.stream, W, ldw, n_rows, p.d_in, p.chan_scale, norms);
    else
        hipLaunchKernelGGL(k_row_norms_vec<1>, grid, dim3(CF_THREADS), 0, p.stream, W, ldw, n_rows, p.d_in, p.chan_scale, norms);
    *err = hipGetLastError();
    return true;
}

// ---------------------------------------------------------------------------------------------
// Calibration of up to CAL_MAX_BATCH matrices in one pair of launches.
// Step 1: one workgroup of 8 waves per chunk of CAL_ROWS consecutive rows of one matrix.  It first computes the norms of
// its rows (slab sums in LDS, to the bit those of the encoders: the head rows are fetched from memory once), then its waves sum
// |z_k| over the chunk's rows, row by row, in fp64, and write one partial sum per pair; CalUnits deals out the slabs.  A
// small matrix is as long as one wave's chain: 256 x 2048, the only launch of 32 workgroups, 20.4 us with a wave per slab, 12.2
// with shared slabs; 1024 head rows of 4096 columns 24.3 -> 16.1.  What is left is some 30 of 51 us of issue for a 7B layer (fp64
// for the most part) and waiting.
// Step 2: per pair, the partial sums added up, then Eq. 1.
// ---------------------------------------------------------------------------------------------
struct CalMat {
    const void *W;
    int64_t ldw;
    const float *chan_scale;
    const int8_t *signs;
    double *partial;                      // n_chunks x (d_in / 2) partial sums
    float *sigma_out;
    int n_rows, d_in, n_slabs, n_chunks;
    float sigma_default;
};
struct CalBatch {
    CalMat m[CAL_MAX_BATCH];
    int chunk_begin[CAL_MAX_BATCH + 1];   // first step-1 workgroup of each matrix
    int fin_begin[CAL_MAX_BATCH + 1];     // first step-2 workgroup of each matrix
    int n;
    float inv_sqrt_block;
};

// acc[k] += |(y[2k], y[2k + 1])|, the square root exact to a few fp64 roundings: the fp32 one (2^-22) and two Newton steps
// (2^-44, then below 2^-53).  Where one of a wave's squares is outside the range of normal fp32, zero included, the library's
// square root.  (So always in a slab that the row ends in, whose idle lanes hold zeros.  Left out of the test, or at work on other
// columns, 48 x 13888 took 32.3 us in place of 33.0, but 4096 x 4096 12.6 in place of 12.4.)  The squares of fp32 are exact in fp64, so the fused sum is rounded as a separate one.
//   The eight chains are free of branches between them: with a test per pair they ran one after the other (4096 x 4096 bf16, this
// launch 15.0 -> 14.4 us).
__device__ __forceinline__ void add_magnitudes(double (&acc)[8], const float (&y)[16]) {
    double a[8];
    float af[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double y0 = (double)y[2 * k], y1 = (double)y[2 * k + 1];
        a[k] = __builtin_fma(y1, y1, y0 * y0);
        af[k] = (float)a[k];
    }
    float least = af[0], most = af[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) {
        least = fminf(least, af[k]);
        most = fmaxf(most, af[k]);
    }
    if (__ballot(!(least >= 1.0e-36f && most <= 1.0e36f)) != 0ull) {
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += sqrt(a[k]);
        return;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float rf = __builtin_amdgcn_rsqf(af[k]);
        const double half = (double)(0.5f * rf);
        double s = (double)(af[k] * rf);
        s = __builtin_fma(__builtin_fma(-s, s, a[k]), half, s);
        acc[k] += __builtin_fma(__builtin_fma(-s, s, a[k]), half, s);
    }
}

// How the waves of a workgroup share its slabs: eight at a time a wave each, and of the rest S waves share a slab's 8 rows, so
// that (nearly) all have some; their sums meet in LDS.  With 11 slabs a wave each, three waves did two slabs where the others
// did one, and a launch is as long as its longest chain: seven matrices of a 7B layer 58.5 -> 51.2 us by the trace, of which these shares,
// scales once per slab and rows requested together in the norms are a part (4096 x 4096 alone 14.4 -> 12.5).
struct CalUnits {
    int whole, rest, shift;                                     // slabs of a wave each, slabs that 1 << shift waves share
    __device__ __forceinline__ explicit CalUnits(int n_slabs)
        : whole(n_slabs & ~(CAL_WAVES - 1)), rest(n_slabs & (CAL_WAVES - 1)), shift(rest > 4 || rest == 0 ? 0 : rest > 2 ? 1 : rest > 1 ? 2 : 3) {}
    __device__ __forceinline__ int count() const { return whole + (rest << shift); }
    // unit u: its slab, and its rows of [row0, row1)
    __device__ __forceinline__ int slab(int u) const { return u < whole ? u : whole + ((u - whole) >> shift); }
    __device__ __forceinline__ void rows(int u, int row0, int row1, int &from, int &to) const {
        const int s = u < whole ? 0 : shift;
        from = row0 + (u & ((1 << s) - 1)) * (CAL_ROWS >> s);   // whole is a multiple of 8
        to = min(row1, from + (CAL_ROWS >> s));
    }
};

template <int DTYPE, int B>
__global__ __launch_bounds__(CAL_THREADS) void k_calibrate_partial(CalBatch bt) {
    __shared__ double norm_part[CAL_ROWS * FUSED_NORM_MAX_SLABS];
    __shared__ float norm_row[CAL_ROWS];
    __shared__ double shared_acc[CAL_WAVES][8][WAVE];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int mi = 0;
    while (mi + 1 < bt.n && (int)blockIdx.x >= bt.chunk_begin[mi + 1]) ++mi;
    const CalMat &M = bt.m[mi];
    Problem p;
    p.d_in = M.d_in;
    p.chan_scale = M.chan_scale;
    p.signs = M.signs;
    const void *__restrict__ W = M.W;
    const int64_t ldw = M.ldw;
    const int n_rows = M.n_rows, n_slabs = M.n_slabs;
    double *__restrict__ partial = M.partial;
    const int chunk = (int)blockIdx.x - bt.chunk_begin[mi];
    const int row0 = chunk * CAL_ROWS, row1 = min(n_rows, row0 + CAL_ROWS);
    const CalUnits units(n_slabs);
    for (int unit = wid; unit < units.count(); unit += CAL_WAVES) {
        const int slab = units.slab(unit);
        int from, to;
        units.rows(unit, row0, row1, from, to);
        const int c = slab * CSLAB + 16 * lane, at = c < p.d_in ? c : 0;
        float sc[16];
        Problem unsigned_scales = p;
        unsigned_scales.signs = nullptr;
        load_signed_scales(sc, unsigned_scales, at);
        auto sums = [&](auto together) __attribute__((always_inline)) {
            constexpr int R = decltype(together)::value;        // rows requested together
#pragma unroll 1
            for (int row = from; row < to; row += R) {
                RawRow<DTYPE> raw[R];
#pragma unroll
                for (int r = 0; r < R; ++r) load_raw_row<DTYPE>(raw[r], W, (int64_t)min(row + r, to - 1) * ldw, at);
                double s2[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {                   // the sums of slab_sum_of_squares(), to the bit
                    float w[16];
                    widen_raw_row<DTYPE>(w, raw[r]);
                    s2[r] = 0.0;
#pragma unroll
                    for (int e = 0; e < 16; ++e) s2[r] = add_square(s2[r], w[e] * sc[e]);
                    s2[r] = c < p.d_in ? s2[r] : 0.0;
                }
                auto put = [&](int r, double sum) {
                    if (row + r < to) norm_part[(row + r - row0) * n_slabs + slab] = sum;
                };
                if constexpr (R == 4) {
                    const double sum = wave_sum_4(s2);
                    if ((lane & 15) == 0) put(lane >> 4, sum);
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double sum = wave_sum(s2[r]);
                        if (lane == 0) put(r, sum);
                    }
                }
            }
        };
        // No more than the unit has, one row of a slab that eight waves share, two of one that four do: with four bf16 rows whatever
        // the unit, 100 x 512 took 7.4 us by the trace, 6.4 so; 1000 x 2048 10.4, 9.0.
        if (to - from == 1) sums(std::integral_constant<int, 1>{});
        else if (DTYPE == 0 || to - from == 2) sums(std::integral_constant<int, 2>{});
        else sums(std::integral_constant<int, 4>{});
    }
    __syncthreads();
    if ((int)threadIdx.x < row1 - row0) norm_row[threadIdx.x] = row_norm_from_slab_sums(norm_part, threadIdx.x, 0, n_slabs);
    __syncthreads();
    const LaneSigns<B> ls(lane);
    const float unit_factor = ls.parity * bt.inv_sqrt_block;
    double acc[8];
    for (int unit = wid; unit < units.count(); unit += CAL_WAVES) {
        const int slab = units.slab(unit);
        int from, to;
        units.rows(unit, row0, row1, from, to);
        const int col0 = slab * CSLAB + 16 * slab_pos(lane);
        const bool active = col0 < p.d_in;
        const int c = active ? col0 : 0;
        float sc[16];
        load_signed_scales(sc, p, c);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = 0.0;
        RawRow<DTYPE> next;
        if (from < to) load_raw_row<DTYPE>(next, W, (int64_t)from * ldw, c);
#pragma unroll 1
        for (int row = from; row < to; ++row) {
            const RawRow<DTYPE> raw = next;
            if (row + 1 < to) load_raw_row<DTYPE>(next, W, (int64_t)(row + 1) * ldw, c);
            float y[16];
            widen_raw_row<DTYPE>(y, raw);
#pragma unroll
            for (int e = 0; e < 16; ++e) y[e] = y[e] * sc[e];
            divide_by_norm(y, __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(norm_row[row - row0]))));
            fwht_wave<B>(y, ls);
#pragma unroll
            for (int e = 0; e < 16; ++e) y[e] = y[e] * unit_factor;
            add_magnitudes(acc, y);
        }
        if ((unit < units.whole || units.shift == 0) && active) {
            double *dst = partial + (int64_t)chunk * (p.d_in >> 1) + (c >> 1);
#pragma unroll
            for (int k = 0; k < 8; ++k) dst[k] = acc[k];
        }
    }
    if (units.shift == 0) return;                               // the same for the whole workgroup
    if (wid < units.rest << units.shift) {                      // whose last unit was whole + wid
#pragma unroll
        for (int k = 0; k < 8; ++k) shared_acc[wid][k][lane] = acc[k];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < units.rest * 8 * WAVE; i += CAL_THREADS) {
        const int sl = i / (8 * WAVE), l = (i & (8 * WAVE - 1)) >> 3, k = i & 7;     // consecutive threads: consecutive pairs of a lane
        const int col0 = (units.whole + sl) * CSLAB + 16 * slab_pos(l);
        if (col0 >= p.d_in) continue;
        const int first = sl << units.shift;
        double s = shared_acc[first][k][l];
        for (int q = 1; q < 1 << units.shift; ++q) s += shared_acc[first + q][k][l];
        partial[(int64_t)chunk * (p.d_in >> 1) + (col0 >> 1) + k] = s;
    }
}

// CF_PAIRS pairs per workgroup, CF_GROUPS threads per pair: each adds a consecutive run of the chunks, the runs' sums are
// added in order.  Bound by memory latency: with one thread per pair a matrix of 2048 pairs was 8 workgroups that each made
// eight round trips (4096 x 4096, 128 chunks: 6.7 us, so 2.8).
constexpr int CF_PAIRS = 32, CF_GROUPS = CF_THREADS / CF_PAIRS;
__global__ __launch_bounds__(CF_THREADS) void k_calibrate_finish(CalBatch bt) {
    __shared__ double sums[CF_GROUPS][CF_PAIRS];
    int mi = 0;
    while (mi + 1 < bt.n && (int)blockIdx.x >= bt.fin_begin[mi + 1]) ++mi;
    const CalMat &M = bt.m[mi];
    const int n_pairs = M.d_in >> 1, n_chunks = M.n_chunks;
    const double *__restrict__ partial = M.partial;
    const int lp = threadIdx.x % CF_PAIRS, group = threadIdx.x / CF_PAIRS;
    const int k = ((int)blockIdx.x - bt.fin_begin[mi]) * CF_PAIRS + lp;
    const int per = (n_chunks + CF_GROUPS - 1) / CF_GROUPS;
    const int end = min(n_chunks, (group + 1) * per);
    double acc = 0.0;
    if (k < n_pairs) {
        int q = group * per;
        for (; q + 16 <= end; q += 16) {                        // 16 loads in flight, added in chunk order
            double v[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) v[t] = partial[(int64_t)(q + t) * n_pairs + k];
#pragma unroll
            for (int t = 0; t < 16; ++t) acc += v[t];
        }
        for (; q < end; ++q) acc += partial[(int64_t)q * n_pairs + k];
    }
    sums[group][lp] = acc;
    __syncthreads();
    if (group != 0 || k >= n_pairs) return;
#pragma unroll
    for (int g = 1; g < CF_GROUPS; ++g) acc += sums[g][lp];
    const double sqrt_half_pi = 1.2533141373155002512078826424055;
    const float s = (float)((acc / (double)M.n_rows) / sqrt_half_pi);
    M.sigma_out[k] = (s > 0.0f) ? s : M.sigma_default;
}

bool fused_norms_supported(const Problem &p) { return (p.d_in + 1023) / 1024 <= FUSED_NORM_MAX_SLABS; }

size_t calibrate_partial_bytes(int d_in, int n_rows) {
    const size_t n_chunks = (size_t)(n_rows + CAL_ROWS - 1) / CAL_ROWS;
    return n_chunks * (size_t)(d_in / 2) * sizeof(double);
}

template <int DTYPE, int B> static hipError_t launch_cal(const CalBatch &bt, hipStream_t stream) {
    hipLaunchKernelGGL((k_calibrate_partial<DTYPE, B>), dim3(bt.chunk_begin[bt.n]), dim3(CAL_THREADS), 0, stream, bt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_calibrate_finish, dim3(bt.fin_begin[bt.n]), dim3(CF_THREADS), 0, stream, bt);
    return hipGetLastError();
}

template <int DTYPE> static hipError_t launch_cal_d(const CalBatch &bt, int block, hipStream_t stream) {
    switch (block) {
        case 64: return launch_cal<DTYPE, 64>(bt, stream);
        case 128: return launch_cal<DTYPE, 128>(bt, stream);
        case 256: return launch_cal<DTYPE, 256>(bt, stream);
        case 512: return launch_cal<DTYPE, 512>(bt, stream);
        case 1024: return launch_cal<DTYPE, 1024>(bt, stream);
        default: return hipErrorNotSupported;
    }
}

bool fast_calibrate_supported(const void *W, int dtype, int64_t ldw, const Problem &p) {
    const int unit = p.block > 16 ? p.block : 16;
    return p.d_in % unit == 0 && p.block >= 64 && fused_norms_supported(p) && front_alignment_ok(W, dtype, ldw, p);
}

// n <= CAL_MAX_BATCH matrices, two launches in all; the kernels compute the head rows' norms themselves.  The caller
// has checked every item with fast_calibrate_supported().
hipError_t launch_calibrate_batch_fast(const CalItem *items, int n, int dtype, int block, hipStream_t stream) {
    if (n < 1 || n > CAL_MAX_BATCH) return hipErrorNotSupported;
    CalBatch bt;
    int64_t chunks = 0, fin = 0;
    // The matrices of the longest rows first: their workgroups take longest, and begun last they ran on alone (a 7B layer, the
    // down projection with its 11 slabs a row last: 62.4 us, so 51.0).  The order inside a launch changes no result.
    int order[CAL_MAX_BATCH];
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order, order + n, [&](int a, int b) { return items[a].d_in > items[b].d_in; });
    for (int i = 0; i < n; ++i) {
        const CalItem &it = items[order[i]];
        CalMat &M = bt.m[i];
        M.W = it.W;
        M.ldw = it.ldw;
        M.chan_scale = it.chan_scale;
        M.signs = it.signs;
        M.partial = it.partial;
        M.sigma_out = it.sigma_out;
        M.n_rows = it.n_rows;
        M.d_in = it.d_in;
        M.n_slabs = (it.d_in + CSLAB - 1) / CSLAB;
        M.n_chunks = (it.n_rows + CAL_ROWS - 1) / CAL_ROWS;
        M.sigma_default = (float)(1.0 / std::sqrt((double)it.d_in));
        bt.chunk_begin[i] = (int)chunks;
        bt.fin_begin[i] = (int)fin;
        chunks += M.n_chunks;
        fin += (it.d_in / 2 + CF_PAIRS - 1) / CF_PAIRS;
        if (chunks > 0x3fffffff || fin > 0x3fffffff) return hipErrorNotSupported;
    }
    for (int i = n; i <= CAL_MAX_BATCH; ++i) {
        bt.chunk_begin[i] = (int)chunks;
        bt.fin_begin[i] = (int)fin;
    }
    for (int i = n; i < CAL_MAX_BATCH; ++i) bt.m[i] = bt.m[0];
    bt.n = n;
    bt.inv_sqrt_block = (float)(1.0 / std::sqrt((double)block));
    return dtype == 0 ? launch_cal_d<0>(bt, block, stream) : launch_cal_d<1>(bt, block, stream);
}

hipError_t launch_calibrate_fast(const void *W, int dtype, int64_t ldw, int n_rows, const Problem &p, double *partial,
                                 float *sigma_out) {
    const CalItem it{W, ldw, p.chan_scale, p.signs, partial, sigma_out, n_rows, p.d_in};
    return launch_calibrate_batch_fast(&it, 1, dtype, p.block, p.stream);
}

}  // namespace qamw
