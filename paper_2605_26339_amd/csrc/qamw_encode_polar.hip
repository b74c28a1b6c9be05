// Polar-baseline encoder (Sec. 3 "Polar Baseline"): the QAM-W front half, then amplitude and phase
// of every pair quantised independently instead of a joint nearest-codeword search.
//
// Front half exactly as the joint encoders (a wave owns one row's slab of 1024 columns, 8 pairs per
// lane, everything in registers).  Per pair x = (x0, x1):
//   amplitude index = number of thresholds below |x|, thresholds at the midpoints of neighbouring
//                     Lloyd-Max levels; decided on squares, a2 = fma(x1, x1, x0 x0) against
//                     T_i = t_i^2, by binary search over the sorted thresholds (no square root);
//   phase index     = the bin [2kh, 2(k+1)h), h = pi/Np, that holds atan2(x1, x0) taken in
//                     [0, 2pi): the half-plane by the sign of x1, then binary search with the
//                     sign of the cross product against the boundary directions (cos 2kh, sin 2kh)
//                     (no arctangent).  The origin has phase bin 0.
// Index = amplitude index * Np + phase index, packed like the joint code, so the decoder is the
// joint decoder with the 2^B-entry table {level_ia * (cos, sin)((2 ip + 1) h)}.
#include <algorithm>

#include "qamw_front.hpp"
#include "qamw_polar_cells.hpp"

namespace qamw {

constexpr int PF_THREADS = 512;
constexpr int PF_WAVES = PF_THREADS / WAVE;
constexpr int PSLAB = 1024;
constexpr int PF_MAX_LEVELS = 64;      // amplitude levels
constexpr int PF_MAX_BINS = 4096;      // phase bins
constexpr int PF_MAX_ROWS = 32;        // rows of a workgroup
constexpr int PF_ITEMS = 48;           // (row, slab) items of a workgroup in a large launch
constexpr int PF_CUS = 256;
constexpr int PF_MAX_ITEMS = 64;       // (row, slab) items of a workgroup, unless one row has more
typedef uint32_t lds_u32x3_t __attribute__((ext_vector_type(3)));
constexpr uint32_t PF_AMP_BASE = (127 - 10) << 5;
constexpr uint32_t PF_LUT_AT = 4 * (PF_MAX_LEVELS + 4) + 8 * PF_MAX_ITEMS + 4 * PF_MAX_ROWS;
constexpr uint32_t PF_DIR_AT = PF_LUT_AT + 8 * PF_AMP_CELLS + 2 * 16 * PF_PHASE_CELLS + 8;   // LDS before the directions

// A workgroup of 8 waves owns `wg_rows` consecutive rows and takes them `rows` at a time: first the slab sums of the first step's
// (row, slab) items, dealt to the waves, then -- after the barrier the table set-up needs anyway -- the items once more, in
// slab-major order, each wave a consecutive share of them, and with each the slab sum of the same item of the next step.  So every
// slab is summed once (a workgroup of four consecutive items summed each row again for each of its items: 11 slabs per row, 3 to 5
// times), and a wave loads, divides and combines the scales, signs and gains of a slab once for all rows of a step.
//   Bound by vector-ALU issue (about 250 instructions of the front half for a wave's 512 pairs, 100 of the slab sum, and per pair
// some 50 of the two binary searches or 27 with the lookup tables), so the lane's pairs go side by side.  4096 x 11008 bf16 at 5 + 6
// bits, 90 MB read, us a call: 115 -> 84 with the slabs summed once, 74 with byte tables that say where the searches would be one
// step before their end, 72 with workgroups that stay for two steps (the second one's norms cost no memory round trips, and the
// tables are made half as often), 66 with entries that hold what is tested and the code (the norms of the second step are 6 of
// that).  11008 x 4096 at 4 + 4 66.5 -> 60, 14336 x 4096 fp32 95 -> 86, 4096 x 4096 fp32 at 3 + 4 36 -> 31 of late.
// (The next item's weights requested ahead: the same.)
template <int DTYPE, int B>
__global__ __launch_bounds__(PF_THREADS) __attribute__((amdgpu_waves_per_eu(4)))   // two workgroups per CU
void k_encode_polar(const void *__restrict__ W, int64_t ldw, Problem p, const float *__restrict__ levels, int bits_a, int bits_p,
                    const float *__restrict__ norms_in, float *__restrict__ norms_out, uint8_t *__restrict__ packed, int n_slabs, int rows,
                    int wg_rows) {
    // LDS: thr2[i] = (midpoint of levels i-1, i)^2, i >= 1, and infinity; the slab sums [row][slab]; the rows' norms; the lookup
    // tables and whether they serve; then the Np boundary directions (cos, sin)(2 k h), and the first again
    constexpr uint32_t THR_AT = 0, PART_AT = 4 * (PF_MAX_LEVELS + 4), NORM_AT = PART_AT + 8 * PF_MAX_ITEMS, DIR_AT = PF_DIR_AT;
    constexpr uint32_t AMP_AT = PF_LUT_AT, PHASE_AT = AMP_AT + 8 * PF_AMP_CELLS, NO_LUT_AT = PHASE_AT + 2 * 16 * PF_PHASE_CELLS;
    static_assert(AMP_AT == NORM_AT + 4 * PF_MAX_ROWS && AMP_AT % 16 == 0 && DIR_AT == NO_LUT_AT + 8, "layout");
    const int Na = 1 << bits_a, Np = 1 << bits_p;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wg_row0 = (int)blockIdx.x * wg_rows, wg_end = min(wg_row0 + wg_rows, p.d_out);
    const int first_rows = min(rows, wg_end - wg_row0);         // of the first step
    const int pos = slab_pos(lane);
    // A slab's scales with their signs and its first column: kept while the wave's items are of that slab.
    int c = 0, cur_slab = -1;
    bool active = false;
    float sc[16], g[8];
    auto at_slab = [&](int slab) __attribute__((always_inline)) {
        cur_slab = slab;
        const int col0 = slab * PSLAB + 16 * pos;
        active = col0 < p.d_in;
        c = active ? col0 : 0;
        load_signed_scales(sc, p, c);
    };
    // the slab's sum of squares of row dr of the next step: that of slab_sum_of_squares() to the bit, since a sign is
    // nothing to a square and the butterfly of wave_sum() meets the same pairs in slab_pos()'s order
    auto put_sum = [&](const RawRow<DTYPE> &raw, int dr, int slab) __attribute__((always_inline)) {
        float w[16];
        widen_raw_row<DTYPE>(w, raw);
        double s2 = 0.0;
#pragma unroll
        for (int e = 0; e < 16; ++e) s2 = add_square(s2, w[e] * sc[e]);
        s2 = wave_sum(active ? s2 : 0.0);
        if (lane == 0) lds_write<double>(PART_AT + 8 * (dr * n_slabs + slab), s2);
    };
    // norms_in == NULL: the workgroup computes its rows' norms (and writes them out)
    if (norms_in == nullptr) {
        for (int t = wid; t < first_rows * n_slabs; t += PF_WAVES) {
            const int dr = t / n_slabs, slab = t - dr * n_slabs;
            const double s2 = slab_sum_of_squares<DTYPE>(W, (int64_t)(wg_row0 + dr) * ldw, slab, p, lane);
            if (lane == 0) lds_write<double>(PART_AT + 8 * t, s2);
        }
    }
    for (int i = threadIdx.x; i < Na; i += PF_THREADS) {
        const float t = (i > 0) ? 0.5f * (levels[i - 1] + levels[i]) : 0.0f;
        lds_write<float>(THR_AT + 4 * i, t * t);
    }
    for (int k = threadIdx.x; k < Np; k += PF_THREADS) {
        float sn, cs;
        sincospif(2.0f * (float)k / (float)Np, &sn, &cs);      // the angle 2 k h = pi * (2k / Np), argument exact
        lds_write<lds_f32x2_t>(DIR_AT + 8 * k, lds_f32x2_t{cs, sn});
    }
    // the workgroup's part of the items (all of them unless a long row is shared by several)
    const PolarPart mine = polar_part((wg_end - wg_row0) * n_slabs, (int)blockIdx.y, (int)gridDim.y, Np);
    const bool want_lut = mine.tables;
    if (threadIdx.x == 0) {
        lds_write<float>(THR_AT + 4 * Na, __builtin_inff());
        lds_write<lds_f32x2_t>(DIR_AT + 8 * Np, lds_f32x2_t{1.0f, 0.0f});
        lds_write<uint32_t>(NO_LUT_AT, want_lut ? 0u : 1u);
    }
    __syncthreads();
    if (want_lut) {
        // thresholds below v, the table taken as sorted (checked: thread i looks at the i-th)
        auto below = [&](float v) {
            int n = 0;
            for (int step = Na >> 1; step; step >>= 1) n = lds_read<float>(THR_AT + 4 * (n + step)) < v ? n + step : n;
            return n;
        };
        const uint32_t cell = threadIdx.x;                      // one each
        static_assert(PF_AMP_CELLS == PF_THREADS, "a cell per thread");
        const float lo = cell ? __uint_as_float((PF_AMP_BASE + cell) << 18) : 0.0f;
        const float hi = cell + 1 < PF_AMP_CELLS ? __uint_as_float((PF_AMP_BASE + cell + 1) << 18) : __builtin_inff();
        const int base = below(lo);
        const bool sorted = (int)cell < 2 || (int)cell >= Na || lds_read<float>(THR_AT + 4 * cell) > lds_read<float>(THR_AT + 4 * (cell - 1));
        if (below(hi) > base + 1 || !sorted) lds_write<uint32_t>(NO_LUT_AT, 1u);
        // the threshold that may lie in the cell, and the code of the level below it
        lds_write<lds_u32x2_t>(AMP_AT + 8 * cell, lds_u32x2_t{__float_as_uint(lds_read<float>(THR_AT + 4 + 4 * base)), (uint32_t)base << bits_p});
        // Phase cells of the upper half plane, then of the lower; boundaries of the half plane certainly passed: place > the cell's end
        static_assert(2 * PF_PHASE_CELLS == PF_THREADS, "a cell per thread");
        const float end = (float)((cell & (PF_PHASE_CELLS - 1)) + 1) * (2.0f / PF_PHASE_CELLS) - 1.0f + 1e-5f;
        int n = 0;
        for (int step = Np >> 2; step; step >>= 1) {
            const lds_f32x2_t b = lds_read<lds_f32x2_t>(DIR_AT + 8 * (n + step));
            n = b[0] / (fabsf(b[0]) + fabsf(b[1])) > end ? n + step : n;
        }
        n += cell < PF_PHASE_CELLS ? 0 : Np >> 1;
        const lds_f32x2_t b = lds_read<lds_f32x2_t>(DIR_AT + 8 + 8 * n);
        lds_write<lds_u32x4_t>(PHASE_AT + 16 * cell, lds_u32x4_t{__float_as_uint(b[0]), __float_as_uint(b[1]), (uint32_t)n, 0u});
    }
    auto put_norms = [&](int row0, int n_rows) {
        const int dr = threadIdx.x;
        if (dr >= n_rows) return;
        float r;
        if (norms_in == nullptr) {
            double s2 = 0.0;                                    // in slab order, as row_norm_from_slab_sums()
            for (int s = 0; s < n_slabs; ++s) s2 += lds_read<double>(PART_AT + 8 * (dr * n_slabs + s));
            r = (float)sqrt(s2);
            if (blockIdx.y == 0) norms_out[row0 + dr] = r;
        } else {
            r = norms_in[row0 + dr];
        }
        lds_write<float>(NORM_AT + 4 * dr, r);
    };
    put_norms(wg_row0, first_rows);
    __syncthreads();

    const bool lut = lds_read<uint32_t>(NO_LUT_AT) == 0u;
    const LaneSigns<B> ls(lane);
    const float unit = ls.parity * p.inv_sqrt_block;
    int odd = 0;
#pragma unroll 1
    for (int row0 = wg_row0; row0 < wg_end; row0 += rows, odd ^= 1) {
        if (row0 > wg_row0) {
            __syncthreads();                                    // the step's sums are there, the norms of the last one are done with
            put_norms(row0, min(rows, wg_end - row0));
            __syncthreads();
        }
        const int n_rows = min(rows, wg_end - row0), next_rows = norms_in == nullptr ? min(rows, wg_end - row0 - rows) : 0;
        // Consecutive shares; in several steps as even as can be, the larger ones to other waves in every other step, and in a single
        // one of few items of a size, which seldom begin with a slab's last.
        const int from = gridDim.y > 1 ? mine.from : 0, n_items = gridDim.y > 1 ? mine.to - mine.from : n_rows * n_slabs;
        auto share = [&](int w) {
            return from + (wg_rows > rows ? (w * n_items + odd * (PF_WAVES - 1)) / PF_WAVES : min(n_items, w * ((n_items + PF_WAVES - 1) / PF_WAVES)));
        };
        const int first = share(wid), last = share(wid + 1);
        for (int item = first; item < last; ++item) {
            const int slab = item / n_rows, dr = item - slab * n_rows, row = row0 + dr;
            if (slab != cur_slab) {
                at_slab(slab);
                load_pair_gains(g, p, c);
            }
            // the same slab of a row of the next step, for its norm
            RawRow<DTYPE> ahead;
            const bool have_ahead = dr < next_rows;

            // ---------------- front half: x_k = (F S (W D_s / r))_pair k / sigma_k, in registers
            RawRow<DTYPE> raw;
            load_raw_row<DTYPE>(raw, W, (int64_t)row * ldw, c);
            if (have_ahead) load_raw_row<DTYPE>(ahead, W, (int64_t)(row + rows) * ldw, c);
            float x[16];
            widen_raw_row<DTYPE>(x, raw);
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = x[e] * sc[e];       // sign included: a sign commutes with every rounding below
            divide_by_norm(x, lds_read<float>(NORM_AT + 4 * (row - row0)));
            fwht_wave<B>(x, ls);
            // Two multiplications also where 1/sqrt(B) is a power of two: y = t / sqrt(B) may be rounded to 0 below the smallest normal
            // number, and the phase of a pair on an axis is not that of one beside it, whatever the gain.
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = x[e] * unit * g[e >> 1];

            // ---------------- amplitude level and phase bin of the lane's 8 pairs
            float a2[8];
            bool upper[8];                                          // angle in [pi, 2 pi)
            unsigned idx[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float x0 = x[2 * k], x1 = x[2 * k + 1];
                a2[k] = __builtin_fmaf(x1, x1, x0 * x0);
                upper[k] = (x1 == 0.0f ? x0 : x1) < 0.0f;
            }
            float most = a2[0], least = a2[0];
#pragma unroll
            for (int k = 1; k < 8; ++k) {
                most = fmaxf(most, a2[k]);
                least = fminf(least, a2[k]);
            }
            if (lut && __ballot(!(most <= PF_LUT_MAX_A2)) == 0ull) {
#pragma unroll
                for (int k0 = 0; k0 < 8; k0 += 4) {                 // four pairs' entries at once are what the registers hold
                    lds_u32x2_t level[4];
                    lds_u32x3_t bin[4];                             // a register for a fourth word would be taken for others, and waited for
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int k = k0 + q;
                        const int cell = min(max((int)(__float_as_uint(a2[k]) >> 18), (int)PF_AMP_BASE), (int)PF_AMP_BASE + PF_AMP_CELLS - 1);
                        level[q] = lds_read<lds_u32x2_t>(AMP_AT - 8 * PF_AMP_BASE + 8 * (uint32_t)cell);
                        const uint32_t at = polar_phase_cell(x[2 * k], x[2 * k + 1], upper[k], [](float s) { return __builtin_amdgcn_rcpf(s); });
                        bin[q] = lds_read<lds_u32x3_t>(PHASE_AT + 16 * at + (upper[k] ? 16 * PF_PHASE_CELLS : 0));
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int k = k0 + q;
                        const float across = __builtin_fmaf(__uint_as_float(bin[q][0]), x[2 * k + 1], -(__uint_as_float(bin[q][1]) * x[2 * k]));
                        idx[k] = level[q][1] + bin[q][2] + (a2[k] > __uint_as_float(level[q][0]) ? (unsigned)Np : 0u) + (across >= 0.0f ? 1u : 0u);
                    }
                }
                if (__ballot(least == 0.0f) != 0ull) {              // the origin: phase bin 0, of level 0
#pragma unroll
                    for (int k = 0; k < 8; ++k) idx[k] = a2[k] == 0.0f ? 0u : idx[k];
                }
            } else {
                unsigned ia[8], ip[8];                              // times 4 and 8: byte offsets into the tables
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    ia[k] = 0;
                    ip[k] = upper[k] ? 8u * (unsigned)(Np >> 1) : 0u;
                }
#pragma unroll 1
                for (unsigned step = 4u * (unsigned)(Na >> 1); step >= 4u; step >>= 1) {
                    float t[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) t[k] = lds_read<float>(THR_AT + ia[k] + step);
#pragma unroll
                    for (int k = 0; k < 8; ++k) ia[k] = (a2[k] > t[k]) ? ia[k] + step : ia[k];   // on the threshold: the lower level
                }
#pragma unroll 1
                for (unsigned step = 8u * (unsigned)(Np >> 2); step >= 8u; step >>= 1) {
                    lds_f32x2_t b[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) b[k] = lds_read<lds_f32x2_t>(DIR_AT + ip[k] + step);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const float cr = __builtin_fmaf(b[k][0], x[2 * k + 1], -(b[k][1] * x[2 * k]));   // sin(angle - 2 cand h) * |x|
                        ip[k] = (cr >= 0.0f) ? ip[k] + step : ip[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) idx[k] = ((ia[k] >> 2) << bits_p) + (a2[k] == 0.0f ? 0u : ip[k] >> 3);
            }

            // ---------------- pack: the lane's 8 fields are exactly `bits` bytes, byte aligned in the row
            if (active) store_fields(packed + (int64_t)row * p.row_bytes, p.row_bytes, p.d_in, c, idx, p.bits);
            if (have_ahead) put_sum(ahead, dr, slab);
        }
    }
}

static bool polar_encode_supported(const Problem &p, int bits_a, int bits_p) {
    const int unit = p.block > 16 ? p.block : 16;
    if (p.d_in % unit || p.block < 64) return false;
    return bits_a >= 0 && bits_p >= 0 && (1 << bits_a) <= PF_MAX_LEVELS && (1 << bits_p) <= PF_MAX_BINS &&
           bits_a + bits_p == p.bits;
}

template <int DTYPE, int B>
static hipError_t launch_pdb(const void *W, int64_t ldw, const Problem &p, const float *levels, int bits_a, int bits_p,
                             float *norms, bool norms_ready, uint8_t *packed) {
    const int n_slabs = (p.d_in + PSLAB - 1) / PSLAB;
    if (!norms_ready && n_slabs > PF_MAX_ITEMS) return hipErrorNotSupported;   // a row's slab sums have to fit the workgroup's list
    // About PF_ITEMS items per workgroup, so that a wave meets a slab several times; fewer while the launch does not give
    // every CU two workgroups (their memory and arithmetic phases alternate), down to one per wave.
    int rows = std::max(1, std::min(PF_MAX_ROWS, PF_ITEMS / n_slabs));
    while (rows > 1 && (p.d_out + rows - 1) / rows < 2 * PF_CUS && (rows + 1) / 2 * n_slabs >= PF_WAVES) rows = (rows + 1) / 2;
    // More than a round of two workgroups per CU: workgroups that stay, and take their rows in steps of about as many, unless an
    // eighth of the chip's would be left without any (2051 x 11008: 411 workgroups of five rows, where 513 of four fill it).
    int wg_rows = rows;
    if ((p.d_out + rows - 1) / rows > 2 * PF_CUS) {
        const int all = (p.d_out + 2 * PF_CUS - 1) / (2 * PF_CUS), steps = (all + rows - 1) / rows;
        if ((p.d_out + all - 1) / all >= 2 * PF_CUS * 7 / 8) {
            wg_rows = all;
            rows = (all + steps - 1) / steps;
        }
    }
    const unsigned blocks = (unsigned)((p.d_out + wg_rows - 1) / wg_rows);
    // Few rows of many slabs: several workgroups share a row, down to an item per wave, each with all slab sums of its own
    // (us by the trace at 5 + 6 bits, bf16, all options, one workgroup a row / so: 16 x 40960 23.4 / 12.1, 64 x 65536 36.0 / 22.1).
    int parts = 1;
    if (wg_rows == 1) parts = std::max(1, std::min((n_slabs + PF_WAVES - 1) / PF_WAVES, 2 * PF_CUS / p.d_out));
    const size_t lds = PF_DIR_AT + 8 * ((size_t)(1 << bits_p) + 1);
    hipLaunchKernelGGL((k_encode_polar<DTYPE, B>), dim3(blocks, (unsigned)parts), dim3(PF_THREADS), lds, p.stream, W, ldw, p, levels, bits_a,
                       bits_p, norms_ready ? norms : nullptr, norms, packed, n_slabs, rows, wg_rows);
    return hipGetLastError();
}

template <int DTYPE>
static hipError_t launch_pd(const void *W, int64_t ldw, const Problem &p, const float *levels, int bits_a, int bits_p,
                            float *norms, bool norms_ready, uint8_t *packed) {
    switch (p.block) {
        case 64: return launch_pdb<DTYPE, 64>(W, ldw, p, levels, bits_a, bits_p, norms, norms_ready, packed);
        case 128: return launch_pdb<DTYPE, 128>(W, ldw, p, levels, bits_a, bits_p, norms, norms_ready, packed);
        case 256: return launch_pdb<DTYPE, 256>(W, ldw, p, levels, bits_a, bits_p, norms, norms_ready, packed);
        case 512: return launch_pdb<DTYPE, 512>(W, ldw, p, levels, bits_a, bits_p, norms, norms_ready, packed);
        case 1024: return launch_pdb<DTYPE, 1024>(W, ldw, p, levels, bits_a, bits_p, norms, norms_ready, packed);
        default: return hipErrorNotSupported;
    }
}

bool polar_encode_launchable(const void *W, int dtype, int64_t ldw, const Problem &p, int bits_a, int bits_p) {
    return polar_encode_supported(p, bits_a, bits_p) && front_alignment_ok(W, dtype, ldw, p) &&
           (reinterpret_cast<uintptr_t>(W) != 0);
}

// Returns hipErrorNotSupported (nothing launched) when the shape or alignment is outside this kernel's range.
hipError_t launch_encode_polar(const void *W, int dtype, int64_t ldw, const Problem &p, const float *levels, int bits_a,
                               int bits_p, float *norms, bool norms_ready, uint8_t *packed) {
    if (!polar_encode_launchable(W, dtype, ldw, p, bits_a, bits_p)) return hipErrorNotSupported;
    return dtype == 0 ? launch_pd<0>(W, ldw, p, levels, bits_a, bits_p, norms, norms_ready, packed)
                      : launch_pd<1>(W, ldw, p, levels, bits_a, bits_p, norms, norms_ready, packed);
}

}  // namespace qamw
