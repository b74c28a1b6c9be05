// Codebook training on the device (Sec. 3.5: Lloyd iterations; a codebook fitted to a checkpoint's own
// pair distribution is the follow-up the paper names) and the samples for it: the normalised pairs the
// encoder quantises.
//
// k_pairs: the encoder's front half (channel scale, row norm, rotation, pair gain), written out instead
// of quantised: bit for bit the points whose nearest codeword qamw_encode stores.
// k_lloyd_assign: every sample to its nearest point by exact fp32 squared distances over the whole
// codebook (lowest index on ties), sums of each cell accumulated in 64-bit fixed point (2^-30), so the
// result does not depend on the order the atomics land in.
// k_lloyd_update: every point to the mean of its cell (an empty cell keeps its point).
// k_cells_lloyd_*: the same iteration for 64 to 2048 points with a cell table (qamw_cells.hpp) made from every iteration's
// points, the sums of a workgroup in LDS first, and the stopping rule on the device, so the host launches ahead.
#include <algorithm>
#include <cmath>

#include "qamw_cells.hpp"
#include "qamw_lloyd_stop.hpp"

namespace qamw {

constexpr int LL_THREADS = 256;
constexpr double LL_SCALE = 1073741824.0;          // 2^30
constexpr float LL_CLAMP = 256.0f;                 // coordinates beyond +-256 enter the sums clamped (2^38 * n < 2^63 for n <= 2^24)

// Accumulators of one assignment pass (in the caller's workspace, after the fp64 codebook).
struct LloydAcc {
    double *cb;                     // K x 2, the points in fp64
    long long *sx, *sy;             // K fixed-point sums
    unsigned long long *cnt;        // K counts
    unsigned long long *err;        // 1: fixed-point sum of squared distances
};

// LDS_SUMS: the cell sums are first accumulated per workgroup in LDS (small codebooks, where thousands of
// samples land on every cell and global atomics on the same address would serialise).
template <bool LDS_SUMS>
__global__ __launch_bounds__(LL_THREADS) void k_lloyd_assign(const float2 *__restrict__ samples, long long n, int K,
                                                             LloydAcc acc) {
    extern __shared__ __align__(16) float2 ll_cb[];
    unsigned long long *lsum = reinterpret_cast<unsigned long long *>(ll_cb + K);   // [3][K]: sx, sy, count (LDS_SUMS only)
    for (int i = threadIdx.x; i < K; i += LL_THREADS) {
        ll_cb[i] = make_float2((float)acc.cb[2 * i], (float)acc.cb[2 * i + 1]);
        if (LDS_SUMS) {
            lsum[i] = 0;
            lsum[K + i] = 0;
            lsum[2 * K + i] = 0;
        }
    }
    __syncthreads();
    double err = 0.0;
    for (long long i = (long long)blockIdx.x * LL_THREADS + threadIdx.x; i < n; i += (long long)gridDim.x * LL_THREADS) {
        const float2 x = samples[i];
        float bd = 3.0e38f;
        int bi = 0;
        for (int k = 0; k < K; ++k) {                           // uniform address: an LDS broadcast
            const float2 c = ll_cb[k];
            const float e0 = x.x - c.x, e1 = x.y - c.y;
            const float d = __builtin_fmaf(e1, e1, e0 * e0);
            if (d < bd) {
                bd = d;
                bi = k;
            }
        }
        const float cx = fminf(fmaxf(x.x, -LL_CLAMP), LL_CLAMP), cy = fminf(fmaxf(x.y, -LL_CLAMP), LL_CLAMP);
        const unsigned long long fx = (unsigned long long)__double2ll_rn((double)cx * LL_SCALE);
        const unsigned long long fy = (unsigned long long)__double2ll_rn((double)cy * LL_SCALE);
        if (LDS_SUMS) {
            atomicAdd(lsum + bi, fx);
            atomicAdd(lsum + K + bi, fy);
            atomicAdd(lsum + 2 * K + bi, 1ull);
        } else {
            atomicAdd(reinterpret_cast<unsigned long long *>(acc.sx + bi), fx);
            atomicAdd(reinterpret_cast<unsigned long long *>(acc.sy + bi), fy);
            atomicAdd(acc.cnt + bi, 1ull);
        }
        err += (double)fminf(bd, 2.0f * LL_CLAMP * LL_CLAMP);
    }
    if (LDS_SUMS) {
        __syncthreads();
        for (int i = threadIdx.x; i < K; i += LL_THREADS) {
            if (lsum[2 * K + i]) {
                atomicAdd(reinterpret_cast<unsigned long long *>(acc.sx + i), lsum[i]);
                atomicAdd(reinterpret_cast<unsigned long long *>(acc.sy + i), lsum[K + i]);
                atomicAdd(acc.cnt + i, lsum[2 * K + i]);
            }
        }
    }
    // one atomic per wave for the error sum
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) err += __shfl_xor(err, s, WAVE);
    if ((threadIdx.x & (WAVE - 1)) == 0) atomicAdd(acc.err, (unsigned long long)__double2ll_rn(err * LL_SCALE));
}

// report[0] = mean squared error of the assignment pass just done
__global__ void k_lloyd_report(long long n, LloydAcc acc, double *report) { report[0] = (double)(*acc.err) / LL_SCALE / (double)n; }

// Either move the points to the means of their cells (move != 0; an empty cell keeps its point) or leave them;
// write the fp32 codebook; clear the sums for the next pass.
__global__ __launch_bounds__(LL_THREADS) void k_lloyd_update(int K, LloydAcc acc, int move, float *codebook_f32) {
    const int i = blockIdx.x * LL_THREADS + threadIdx.x;
    if (i == 0) *acc.err = 0;
    if (i < K) {
        const unsigned long long c = acc.cnt[i];
        if (move && c > 0) {
            acc.cb[2 * i] = (double)acc.sx[i] / LL_SCALE / (double)c;
            acc.cb[2 * i + 1] = (double)acc.sy[i] / LL_SCALE / (double)c;
        }
        codebook_f32[2 * i] = (float)acc.cb[2 * i];
        codebook_f32[2 * i + 1] = (float)acc.cb[2 * i + 1];
        acc.sx[i] = 0;
        acc.sy[i] = 0;
        acc.cnt[i] = 0;
    }
}

__global__ __launch_bounds__(LL_THREADS) void k_lloyd_init(int K, LloydAcc acc, const float *codebook_f32) {
    const int i = blockIdx.x * LL_THREADS + threadIdx.x;
    if (i == 0) *acc.err = 0;
    if (i < K) {
        acc.cb[2 * i] = (double)codebook_f32[2 * i];
        acc.cb[2 * i + 1] = (double)codebook_f32[2 * i + 1];
        acc.sx[i] = 0;
        acc.sy[i] = 0;
        acc.cnt[i] = 0;
    }
}

// ------------------------------------------------------------------------------------------------ with a cell table
// Per iteration t, points and sums in buffer t mod 2: k_cells_lloyd_table moves the points to the means of their cells in
// iteration t - 1 and makes the table, k_cells_lloyd_assign assigns every sample and adds to the sums.  After iteration t the
// next launch decides whether to stop; the kernels of later iterations then return at once.
//   What bounds it: two launches that are each mostly latency.  2048 points, 2^20 samples (8 MB): 10.2 + 15.2 us an iteration.
// A copy of the sums per workgroup (10.5 MB, more than the samples), added up by a launch of its own: 9.2 + 13.9 + 7.7; the
// distances to all points took 401.
constexpr int LC_THREADS = 1024;
constexpr int LC_MAX_BLOCKS = 256;                             // one workgroup per CU: a workgroup's sums are 20 bytes per point, each added to the one copy
constexpr int LC_SAMPLES = 4;                                  // of a thread at once
constexpr int LC_AHEAD = 16;                                   // iterations launched before the host looks whether it has stopped
constexpr int LC_DENSE_ABOVE = 16;                             // of a wave's 64 samples
constexpr int lc_side(int K) { return K >= 1024 ? 128 : 64; }

struct LloydCells {
    unsigned long long *sx[2], *sy[2];                         // K fixed-point sums
    float *cb32[2];
    uint2 *table;
    unsigned *cnt[2];
    unsigned long long *err;                                   // [2]
    LloydState *state;
};
static size_t lloyd_cells_bytes(int K) {
    const size_t G = lc_side(K);
    return (size_t)K * 2 * (16 + 8 + 4) + G * G * 8 + 128;
}
static LloydCells lloyd_cells_layout(void *workspace, int K) {
    LloydCells a;
    char *p = static_cast<char *>(workspace);
    auto take = [&](size_t bytes) {
        char *at = p;
        p += bytes;
        return at;
    };
    a.state = reinterpret_cast<LloydState *>(take(64));
    a.err = reinterpret_cast<unsigned long long *>(take(64));
    for (int i = 0; i < 2; ++i) {
        a.sx[i] = reinterpret_cast<unsigned long long *>(take((size_t)K * 8));
        a.sy[i] = reinterpret_cast<unsigned long long *>(take((size_t)K * 8));
        a.cb32[i] = reinterpret_cast<float *>(take((size_t)K * 8));
        a.cnt[i] = reinterpret_cast<unsigned *>(take((size_t)K * 4));
    }
    a.table = reinterpret_cast<uint2 *>(take((size_t)lc_side(K) * lc_side(K) * 8));
    return a;
}

// The caller's points as the points of iteration -1, whose cells are all empty.
__global__ __launch_bounds__(LL_THREADS) void k_cells_lloyd_init(int K, LloydCells a, const float *codebook) {
    const int i = blockIdx.x * LL_THREADS + threadIdx.x;
    if (i < 2 * K) a.cb32[1][i] = codebook[i];
    if (i < K) {
        a.sx[1][i] = 0;
        a.sy[1][i] = 0;
        a.cnt[1][i] = 0;
    }
    if (i == 0) {
        a.err[1] = 0;
        *a.state = lloyd_begin();
    }
}

// The mean squared error of iteration t, and whether it was the last.
__device__ __forceinline__ bool lloyd_stops(const LloydCells &a, long long n, int t, int max_iters, double tol, double &D) {
    const double prev = a.state->D[(t + 1) & 1];
    D = (double)a.err[t & 1] / LL_SCALE / (double)n;
    return (t > 0 && fabs(prev - D) < tol * prev) || t + 1 >= max_iters;
}

// Every workgroup computes all points, each writes its share of them and clears that share of this iteration's sums.  The
// sums of iteration t - 1 are read by this launch alone.  One thread decides whether t - 1 was the last iteration; if so, what
// this launch makes is not looked at.
template <int G>
__global__ __launch_bounds__(CP_THREADS) void k_cells_lloyd_table(int K, float half_per_sum, LloydCells a, long long n, int t, int max_iters, double tol) {
    __shared__ float2 points[2048 + 2048 / 8];                 // a place left out after eight: a thread reads a run of up to eight
    auto place = [](int i) { return i + (i >> 3); };
    const int from = (t + 1) & 1, to = t & 1;
    const int stopped_at = lloyd_seen_by_table(*a.state, t);
    float2 old[CP_PER_THREAD];
    long long sx[CP_PER_THREAD], sy[CP_PER_THREAD];
    unsigned c[CP_PER_THREAD];
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) {
        const int k = min((int)threadIdx.x + CP_THREADS * j, K - 1);
        c[j] = a.cnt[from][k];
        sx[j] = (long long)a.sx[from][k];
        sy[j] = (long long)a.sy[from][k];
        old[j] = reinterpret_cast<const float2 *>(a.cb32[from])[k];
    }
    const bool decides = blockIdx.x == 0 && threadIdx.x == 0;
    if (stopped_at != LC_RUNNING) {
        if (decides) lloyd_table_decides(*a.state, t, false);
        return;
    }
    const int share = max(K / (int)gridDim.x, 1);
#pragma unroll
    for (int j = 0; j < CP_PER_THREAD; ++j) {
        const int k = (int)threadIdx.x + CP_THREADS * j;
        if (k >= K) break;
        const double px = (double)sx[j] / LL_SCALE / (double)c[j], py = (double)sy[j] / LL_SCALE / (double)c[j];
        const float2 p = c[j] > 0 ? make_float2((float)px, (float)py) : old[j];   // an empty cell keeps its point
        points[place(k)] = p;
        if (k / share == (int)blockIdx.x) {
            reinterpret_cast<float2 *>(a.cb32[to])[k] = p;
            a.sx[to][k] = 0;
            a.sy[to][k] = 0;
            a.cnt[to][k] = 0;
        }
    }
    if (decides) {
        a.err[to] = 0;
        double D = 0.0;
        const bool stops = t > 0 && lloyd_stops(a, n, t - 1, max_iters, tol, D);
        a.state->D[from] = D;
        lloyd_table_decides(*a.state, t, stops);
    }
    __syncthreads();
    cells_build_region<G>(cells_points(K, [&](int i) { return points[place(i)]; }), K, half_per_sum, a.table, (int)blockIdx.x);
}

// The records come from memory (L2), four samples' at a time: staging them took as long as the samples of a workgroup do, and
// a table of 112 x 112 cells was all that fitted beside the sums, with 1.1 % of Gaussian samples in cells of six candidates
// while cells were of one width -- a scan of the whole codebook in most waves, against 0.05 % with 128 x 128 (0.001 % with the cells of
// now).  2048 points, 2^20 samples: 23.5 -> 11.5 us.
//   The sums' atomics, three per point and workgroup, are what a workgroup costs whatever its share; see lc_blocks().
template <int G>
__global__ __launch_bounds__(LC_THREADS) void k_cells_lloyd_assign(const float2 *__restrict__ samples, long long n, int K, LloydCells a, int t) {
    // points (at LDS address 0), then the sums: x, y (64 bits), count (32), error (64)
    extern __shared__ __align__(16) float2 lc_lds[];
    constexpr int U = LC_SAMPLES;
    static_assert((G & (G - 1)) == 0, "the mask of the record's offset");
    const int stopped_at = lloyd_seen_by_assignment(*a.state, t);
    const float half = cells_half(a.table);
    const int lane = threadIdx.x & (WAVE - 1);
    const long long stride = (long long)gridDim.x * LC_THREADS;
    long long i = (long long)blockIdx.x * LC_THREADS + threadIdx.x;
    const float2 *cbk = reinterpret_cast<const float2 *>(a.cb32[t & 1]);
    float2 next[U];
    auto request = [&](long long at) {
#pragma unroll
        for (int u = 0; u < U; ++u) next[u] = at + u * stride < n ? samples[at + u * stride] : make_float2(0.0f, 0.0f);
    };
    request(i);
    unsigned long long *sx = reinterpret_cast<unsigned long long *>(lc_lds + K), *sy = sx + K;
    unsigned *cnt = reinterpret_cast<unsigned *>(sy + K);
    unsigned long long &err_sum = *reinterpret_cast<unsigned long long *>(cnt + K);
    for (int k = threadIdx.x; k < K; k += LC_THREADS) {
        lc_lds[k] = cbk[k];
        sx[k] = 0;
        sy[k] = 0;
        cnt[k] = 0;
    }
    if (threadIdx.x == 0) err_sum = 0;
    if (stopped_at != LC_RUNNING) return;
    const float inv_span = cells_inv_span(half), far = cells_far(half);
    __syncthreads();

    double err = 0.0;
    for (; i - lane < n; i += U * stride) {                     // the wave's lanes stay together
        float2 x[U];
        uint2 rec[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = next[u];
            rec[u] = *reinterpret_cast<const uint2 *>(reinterpret_cast<const char *>(a.table) +
                                                      (cells_record_at<G>(x[u].x, x[u].y, inv_span, 0u) & (G * G * 8u - 1u)));   // in range whatever x is
        }
        request(i + U * stride);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool active = i + u * stride < n;
            CellsFour four;
            cells_request(four, rec[u], 0u);
            double best = cells_nearest(four, x[u].x, x[u].y);
            if (__ballot(rec[u].y & CELLS_FIFTH)) best = cells_fifth(rec[u], x[u].x, x[u].y, 0u, best);
            int bi = (int)(cells_offset(best) >> 3);
            float d = cells_distance(best);
            unsigned long long mask = __ballot(active && cells_undecided<true>(rec[u], x[u].x, x[u].y, far));
            // outside the table, or too many candidates: the whole codebook, for many samples at once or one after the other
            if (__popcll(mask) > LC_DENSE_ABOVE) {
                const float x0[1] = {x[u].x}, x1[1] = {x[u].y};
                unsigned found[1];
                nearest_of_all<1, (G == 64 ? 1 : 2), (G == 64 ? 64 : 1024), (G == 64 ? 512 : 2048)>(x0, x1, found, (mask >> lane) & 1u, 0u, K, lane);
                if ((mask >> lane) & 1u) {
                    bi = (int)(found[0] >> 3);
                    d = fminf(exact_dist2(x[u].x, x[u].y, lc_lds[bi]), 3.0e38f);
                }
                mask = 0;
            }
            while (mask) {
                const int at = __ffsll((long long)mask) - 1;
                mask &= mask - 1;
                const float x0 = __shfl(x[u].x, at, WAVE), x1 = __shfl(x[u].y, at, WAVE);
                const int found = wave_exact_scan<(G == 64 ? 64 : 1024), (G == 64 ? 512 : 2048)>(x0, x1, 0u, K, lane);
                if (lane == at) {
                    bi = found;
                    d = fminf(exact_dist2(x0, x1, lc_lds[found]), 3.0e38f);
                }
            }
            if (active) {
                const float cx = fminf(fmaxf(x[u].x, -LL_CLAMP), LL_CLAMP), cy = fminf(fmaxf(x[u].y, -LL_CLAMP), LL_CLAMP);
                atomicAdd(sx + bi, (unsigned long long)__double2ll_rn((double)cx * LL_SCALE));
                atomicAdd(sy + bi, (unsigned long long)__double2ll_rn((double)cy * LL_SCALE));
                atomicAdd(cnt + bi, 1u);
                err += (double)fminf(d, 2.0f * LL_CLAMP * LL_CLAMP);
            }
        }
    }
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) err += __shfl_xor(err, s, WAVE);
    if (lane == 0) atomicAdd(&err_sum, (unsigned long long)__double2ll_rn(err * LL_SCALE));
    __syncthreads();
    // each workgroup begins somewhere else, so that they seldom meet at an address
    unsigned long long *to_x = a.sx[t & 1], *to_y = a.sy[t & 1];
    unsigned *to_n = a.cnt[t & 1];
    for (int i = threadIdx.x; i < K; i += LC_THREADS) {
        const int k = (i + (int)blockIdx.x * WAVE) & (K - 1);
        if (cnt[k] == 0) continue;
        atomicAdd(to_x + k, sx[k]);
        atomicAdd(to_y + k, sy[k]);
        atomicAdd(to_n + k, cnt[k]);
    }
    if (threadIdx.x == 0) atomicAdd(a.err + (t & 1), err_sum);
}

// After iteration t, the last that was launched: if it or one before it was the last, the points of the last assignment.
__global__ __launch_bounds__(LL_THREADS) void k_cells_lloyd_finish(long long n, int K, LloydCells a, int t, int max_iters, double tol, float *codebook) {
    const int i = blockIdx.x * LL_THREADS + threadIdx.x;
    const float points[2] = {i < 2 * K ? a.cb32[0][i] : 0.0f, i < 2 * K ? a.cb32[1][i] : 0.0f};   // on their way meanwhile
    int at = lloyd_seen_by_assignment(*a.state, t);
    if (at == LC_RUNNING) {
        double D;
        if (!lloyd_stops(a, n, t, max_iters, tol, D)) return;
        at = t;
        if (i == 0) a.state->D[t & 1] = D;
    }
    if (i == 0) a.state->last = at;
    if (i < 2 * K) codebook[i] = at & 1 ? points[1] : points[0];
}

// Workgroups of the assignment.  They work in passes of LC_SAMPLES samples a thread, and each adds its sums to the one copy at the
// end.  So from half of the chip on as many as one pass needs; with 2048 points, whose atomics cost more than a pass, two.
//   Us an iteration, both launches and the host's look, 128 / so / 256 workgroups, started from a codebook for such samples and
// (in brackets) from points drawn at random, of which more samples are left to a scan of all points:
//     64 points, 600 000 samples      18.7 / 18.9 / 20.6 (19.0 / 19.0 / 20.4),  2^20 20.7 / 20.9 / 20.9,  2^21 25.1 / 23.5 / 23.5
//     1024 points, 700 000            23.5 / 22.7 / 23.9 (30.0 / 26.1 / 26.3),  2^20 24.4 / 24.6 / 24.6 (34.1 / 28.0 / 28.0)
//     2048 points, 2^20               28.3 / 28.3 / 30.9 (51.9 / 51.9 / 41.1),  1 250 000 30.4 / 29.5 / 31.0 (58.5 / 53.3 / 45.1),
//                  2^21               33.7 / 33.7 / 33.7 (79.8 / 55.3 / 55.3)
// Below half of the chip: 64 points, 2^18 samples 16.9 with 64 workgroups, 17.3 with 128, but 2048 points at random 37.8, 31.0.
static unsigned lc_blocks(int K, long long n) {
    const long long pass = (long long)LC_THREADS * LC_SAMPLES * (K >= 2048 ? 2 : 1);
    const long long want = std::min((n + pass - 1) / pass, (long long)LC_MAX_BLOCKS);
    return (unsigned)std::min(std::max(want, (long long)LC_MAX_BLOCKS / 2), (n + LC_THREADS - 1) / LC_THREADS);
}

template <int G>
static hipError_t run_lloyd_cells(const float *samples, long long n, int K, float *codebook, int max_iters, double tol,
                                  void *workspace, double *mse_out, int *iters_out, hipStream_t stream) {
    const LloydCells a = lloyd_cells_layout(workspace, K);
    // points and sums; and no less than the table's first record, which does not hold indices, can point to
    const size_t lds = std::max((size_t)K * 28 + 8, (size_t)4096 * 8);
    static_assert(2048 * 28 + 8 <= 64 * 1024, "what a workgroup may have without asking");
    const float half_per_sum = cells_half_per_sum(__builtin_ctz((unsigned)K));
    const unsigned kb = (unsigned)((2 * K + LL_THREADS - 1) / LL_THREADS);
    const unsigned blocks = lc_blocks(K, n);
    hipLaunchKernelGGL(k_cells_lloyd_init, dim3(kb), dim3(LL_THREADS), 0, stream, K, a, codebook);
    LloydState s = lloyd_begin();
    for (int t = 0; s.last == LC_RUNNING;) {
        const int until = max_iters - t < LC_AHEAD ? max_iters : t + LC_AHEAD;
        for (; t < until; ++t) {
            hipLaunchKernelGGL(k_cells_lloyd_table<G>, dim3((G / 8) * (G / 8)), dim3(CP_THREADS), 0, stream, K, half_per_sum, a, n, t, max_iters, tol);
            hipLaunchKernelGGL(k_cells_lloyd_assign<G>, dim3(blocks), dim3(LC_THREADS), lds, stream,
                               reinterpret_cast<const float2 *>(samples), n, K, a, t);
        }
        hipLaunchKernelGGL(k_cells_lloyd_finish, dim3(kb), dim3(LL_THREADS), 0, stream, n, K, a, t - 1, max_iters, tol, codebook);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = hipMemcpyAsync(&s, a.state, sizeof s, hipMemcpyDeviceToHost, stream);
        if (e != hipSuccess) return e;
        e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return e;
    }
    if (mse_out) *mse_out = s.D[s.last & 1];
    if (iters_out) *iters_out = s.last + 1;
    return hipSuccess;
}

// With a cell table from 64 points on: with fewer the distances to all of them are sooner computed than a table made.
static bool lloyd_has_cells(int K) { return K >= 64 && K <= 2048; }
size_t lloyd_least_workspace_bytes(int K) { return (size_t)K * (2 * sizeof(double) + 3 * sizeof(long long)) + 64; }
size_t lloyd_workspace_bytes(int K) {
    const size_t least = lloyd_least_workspace_bytes(K);
    return lloyd_has_cells(K) && lloyd_cells_bytes(K) > least ? lloyd_cells_bytes(K) : least;
}

static LloydAcc lloyd_layout(void *workspace, int K) {
    LloydAcc a;
    char *p = static_cast<char *>(workspace);
    a.cb = reinterpret_cast<double *>(p);
    p += (size_t)K * 2 * sizeof(double);
    a.sx = reinterpret_cast<long long *>(p);
    p += (size_t)K * sizeof(long long);
    a.sy = reinterpret_cast<long long *>(p);
    p += (size_t)K * sizeof(long long);
    a.cnt = reinterpret_cast<unsigned long long *>(p);
    p += (size_t)K * sizeof(long long);
    a.err = reinterpret_cast<unsigned long long *>(p);
    return a;
}

// Lloyd iterations with the stopping rule of the CPU trainer: after each assignment the mean squared error D is
// read back; stop when |D_prev - D| < tol * D_prev (from the second assignment on) or after max_iters assignments;
// the points are not moved after the last assignment.  Blocks the host on the stream once per iteration.
hipError_t run_lloyd(const float *samples, long long n, int K, float *codebook, int max_iters, double tol, void *workspace,
                     size_t workspace_bytes, double *mse_out, int *iters_out, hipStream_t stream) {
    if (lloyd_has_cells(K) && workspace_bytes >= lloyd_cells_bytes(K)) {
        if (lc_side(K) == 128) return run_lloyd_cells<128>(samples, n, K, codebook, max_iters, tol, workspace, mse_out, iters_out, stream);
        return run_lloyd_cells<64>(samples, n, K, codebook, max_iters, tol, workspace, mse_out, iters_out, stream);
    }
    const LloydAcc acc = lloyd_layout(workspace, K);
    double *report = reinterpret_cast<double *>(reinterpret_cast<char *>(acc.err) + 16);
    const unsigned kb = (unsigned)((K + LL_THREADS - 1) / LL_THREADS);
    const bool lds_sums = K <= 1024;
    const long long want = (n + LL_THREADS - 1) / LL_THREADS, cap = lds_sums ? 1024 : 4096;
    const unsigned blocks = (unsigned)(want < cap ? (want < 1 ? 1 : want) : cap);
    hipLaunchKernelGGL(k_lloyd_init, dim3(kb), dim3(LL_THREADS), 0, stream, K, acc, codebook);
    double prev = 0.0, D = 0.0;
    int it = 0;
    for (;; ++it) {
        if (lds_sums)
            hipLaunchKernelGGL(k_lloyd_assign<true>, dim3(blocks), dim3(LL_THREADS), (size_t)K * (sizeof(float2) + 24), stream,
                               reinterpret_cast<const float2 *>(samples), n, K, acc);
        else
            hipLaunchKernelGGL(k_lloyd_assign<false>, dim3(blocks), dim3(LL_THREADS), (size_t)K * sizeof(float2), stream,
                               reinterpret_cast<const float2 *>(samples), n, K, acc);
        // the decision to move needs D on the host: read it with the sums still in place, then move or not
        hipLaunchKernelGGL(k_lloyd_report, dim3(1), dim3(1), 0, stream, n, acc, report);
        hipError_t e = hipMemcpyAsync(&D, report, sizeof(double), hipMemcpyDeviceToHost, stream);
        if (e != hipSuccess) return e;
        e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return e;
        const bool stop = (it > 0 && std::fabs(prev - D) < tol * prev) || it + 1 >= max_iters;
        hipLaunchKernelGGL(k_lloyd_update, dim3(kb), dim3(LL_THREADS), 0, stream, K, acc, stop ? 0 : 1, codebook);
        prev = D;
        if (stop) break;
    }
    if (mse_out) *mse_out = D;
    if (iters_out) *iters_out = it + 1;
    hipError_t e = hipStreamSynchronize(stream);
    return e != hipSuccess ? e : hipGetLastError();
}

// ---------------------------------------------------------------------------------------------- pairs
template <int DTYPE, int B>
__global__ __launch_bounds__(LL_THREADS) void k_pairs(const void *__restrict__ W, int64_t ldw, Problem p,
                                                      const float *__restrict__ norms_in, float *__restrict__ norms_out,
                                                      float *__restrict__ pairs, int n_slabs, int n_items, int n_blocks) {
    constexpr int NW = LL_THREADS / WAVE;
    __shared__ double norm_part[2 * FUSED_NORM_MAX_SLABS];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = threadIdx.x >> 6;
    // norms_in == NULL: the workgroup computes the norms of the rows its items touch (and writes them out)
    const bool fused = norms_in == nullptr;
    const int item0 = (fused ? fused_norm_block(blockIdx.x, n_blocks) : (int)blockIdx.x) * NW;
    if (fused) {
        if (item0 < n_items) block_slab_sums<DTYPE, NW>(norm_part, W, ldw, p, item0, n_items, n_slabs, lane, wid);
        __syncthreads();
    }
    const int item = __builtin_amdgcn_readfirstlane(item0 + wid);
    if (item >= n_items) return;
    const int row = item / n_slabs, slab = item - row * n_slabs;
    float rnorm;
    if (fused) {
        rnorm = row_norm_from_slab_sums(norm_part, row, item0, n_slabs);
        if (slab == 0 && lane == 0) norms_out[row] = rnorm;
    } else {
        rnorm = norms_in[row];
    }
    const LaneSigns<B> ls(lane);
    const int pos = slab_pos(lane);
    const int col0 = slab * 1024 + 16 * pos;
    const bool active = col0 < p.d_in;
    const int c = active ? col0 : 0;
    float x[16];
    rotated_unit_row<DTYPE, B>(x, W, (int64_t)row * ldw, c, rnorm, p, ls);
    float g[8];
    if (p.pair_sigma) {
        const float4 *g4 = reinterpret_cast<const float4 *>(p.pair_sigma + (c >> 1));
        float4 a = g4[0], b = g4[1];
        const float sg8[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = 1.0f / sg8[k];                         // IEEE division
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = p.g_default;
    }
    if (active) {
        float4 *dst = reinterpret_cast<float4 *>(pairs + (int64_t)row * p.d_in + c);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            dst[t] = make_float4(x[4 * t] * g[2 * t], x[4 * t + 1] * g[2 * t], x[4 * t + 2] * g[2 * t + 1], x[4 * t + 3] * g[2 * t + 1]);
    }
}

bool pairs_launchable(const void *W, int dtype, int64_t ldw, const Problem &p, const float *pairs) {
    const int unit = p.block > 16 ? p.block : 16;
    return p.d_in % unit == 0 && p.block >= 64 && front_alignment_ok(W, dtype, ldw, p) &&
           (reinterpret_cast<uintptr_t>(pairs) & 15) == 0;
}

template <int DTYPE>
static hipError_t launch_pairs_d(const void *W, int64_t ldw, const Problem &p, float *norms, bool norms_ready, float *pairs) {
    const int n_slabs = (p.d_in + 1023) / 1024;
    const int64_t n_items = (int64_t)p.d_out * n_slabs;
    if (n_items > 0x7fffffff) return hipErrorNotSupported;
    if (!norms_ready && n_slabs > FUSED_NORM_MAX_SLABS) return hipErrorNotSupported;
    static_assert(LL_THREADS / WAVE == 4, "four items per workgroup");
    const int n_blocks = (int)((n_items + 3) / 4);
    const unsigned blocks = (unsigned)(norms_ready ? n_blocks : fused_norm_grid(n_blocks));
    const float *norms_in = norms_ready ? norms : nullptr;
#define QAMW_PAIRS(BB) \
    case BB: hipLaunchKernelGGL((k_pairs<DTYPE, BB>), dim3(blocks), dim3(LL_THREADS), 0, p.stream, W, ldw, p, norms_in, norms, pairs, n_slabs, (int)n_items, n_blocks); break;
    switch (p.block) {
        QAMW_PAIRS(64) QAMW_PAIRS(128) QAMW_PAIRS(256) QAMW_PAIRS(512) QAMW_PAIRS(1024)
        default: return hipErrorNotSupported;
    }
#undef QAMW_PAIRS
    return hipGetLastError();
}

hipError_t launch_pairs(const void *W, int dtype, int64_t ldw, const Problem &p, float *norms, bool norms_ready, float *pairs) {
    if (!pairs_launchable(W, dtype, ldw, p, pairs)) return hipErrorNotSupported;
    return dtype == 0 ? launch_pairs_d<0>(W, ldw, p, norms, norms_ready, pairs) : launch_pairs_d<1>(W, ldw, p, norms, norms_ready, pairs);
}

}  // namespace qamw
