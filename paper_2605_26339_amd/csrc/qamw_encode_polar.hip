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
constexpr uint32_t PF_AMP_BASE = (127 - 10) << 5;
constexpr uint32_t PF_LUT_AT = 4 * (PF_MAX_LEVELS + 4) + 8 * PF_MAX_ITEMS + 4 * PF_MAX_ROWS;
constexpr uint32_t PF_DIR_AT = PF_LUT_AT + PF_AMP_CELLS + PF_PHASE_CELLS + 8;   // LDS before the directions

// A workgroup of 8 waves owns `rows` consecutive rows: first the slab sums of all their (row, slab) items, dealt to the
// waves, then -- after the barrier the table set-up needs anyway -- the items once more, in slab-major order, each wave a
// consecutive share of them.  So every slab is summed once (a workgroup of four consecutive items summed each row again
// for each of its items: 11 slabs per row, 3 to 5 times), and a wave loads, divides and combines the scales, signs and
// gains of a slab once for all rows it has of it.
//   Bound by vector-ALU issue (about 250 instructions of the front half for a wave's 512 pairs, and per pair some 50 of the two
// binary searches or 25 with the lookup tables), so the lane's 8 pairs go side by side: eight table reads in flight per step.
// 4096 x 11008 bf16 at 5 + 6 bits, 90 MB read: 115 -> 80 us with searches, 68 so (333 Gpairs/s); 11008 x 4096 at 4 + 4 73 -> 69.
// (The next item's weights requested ahead: 1 to 3 % slower.)
template <int DTYPE, int B>
__global__ __launch_bounds__(PF_THREADS) void k_encode_polar(const void *__restrict__ W, int64_t ldw, Problem p,
                                                             const float *__restrict__ levels, int bits_a, int bits_p,
                                                             const float *__restrict__ norms_in, float *__restrict__ norms_out,
                                                             uint8_t *__restrict__ packed, int n_slabs, int rows) {
    // LDS: thr2[i] = (midpoint of levels i-1, i)^2, i >= 1, and infinity; the slab sums [row][slab]; the rows' norms; the lookup
    // tables and whether they serve; then the Np boundary directions (cos, sin)(2 k h), and the first again
    constexpr uint32_t THR_AT = 0, PART_AT = 4 * (PF_MAX_LEVELS + 4), NORM_AT = PART_AT + 8 * PF_MAX_ITEMS, DIR_AT = PF_DIR_AT;
    constexpr uint32_t AMP_AT = PF_LUT_AT, PHASE_AT = AMP_AT + PF_AMP_CELLS, NO_LUT_AT = PHASE_AT + PF_PHASE_CELLS;
    static_assert(AMP_AT == NORM_AT + 4 * PF_MAX_ROWS && DIR_AT == NO_LUT_AT + 8, "layout");
    const int Na = 1 << bits_a, Np = 1 << bits_p;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = (int)blockIdx.x * rows, n_rows = min(rows, p.d_out - row0), n_items = n_rows * n_slabs;
    // norms_in == NULL: the workgroup computes its rows' norms (and writes them out)
    if (norms_in == nullptr) {
        for (int t = wid; t < n_items; t += PF_WAVES) {
            const int dr = t / n_slabs, slab = t - dr * n_slabs;
            const double s2 = slab_sum_of_squares<DTYPE>(W, (int64_t)(row0 + dr) * ldw, slab, p, lane);
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
    const PolarPart mine = polar_part(n_items, (int)blockIdx.y, (int)gridDim.y, Np);
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
        lds_write<uint8_t>(AMP_AT + cell, (uint8_t)(4 * base));
        if (cell < PF_PHASE_CELLS) {                            // boundaries of the upper half plane certainly passed: place > the cell's end
            const float end = (float)(cell + 1) * (2.0f / PF_PHASE_CELLS) - 1.0f + 1e-5f;
            int n = 0;
            for (int step = Np >> 2; step; step >>= 1) {
                const lds_f32x2_t b = lds_read<lds_f32x2_t>(DIR_AT + 8 * (n + step));
                n = b[0] / (fabsf(b[0]) + fabsf(b[1])) > end ? n + step : n;
            }
            lds_write<uint8_t>(PHASE_AT + cell, (uint8_t)n);
        }
    }
    if ((int)threadIdx.x < n_rows) {
        const int dr = threadIdx.x;
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
    }
    __syncthreads();

    const bool lut = lds_read<uint32_t>(NO_LUT_AT) == 0u;
    const LaneSigns<B> ls(lane);
    const int pos = slab_pos(lane);
    const float unit = ls.parity * p.inv_sqrt_block;
    const int per = (mine.to - mine.from + PF_WAVES - 1) / PF_WAVES;
    const int first = mine.from + wid * per, last = min(mine.to, first + per);
    int c = 0, cur_slab = -1;
    bool active = false;
    float sc[16], g[8];
    for (int item = first; item < last; ++item) {
        const int slab = item / n_rows, row = row0 + item - slab * n_rows;
        if (slab != cur_slab) {
            cur_slab = slab;
            const int col0 = slab * PSLAB + 16 * pos;
            active = col0 < p.d_in;
            c = active ? col0 : 0;
            load_signed_scales(sc, p, c);
            load_pair_gains(g, p, c);
        }

        // ---------------- front half: x_k = (F S (W D_s / r))_pair k / sigma_k, in registers
        RawRow<DTYPE> raw;
        load_raw_row<DTYPE>(raw, W, (int64_t)row * ldw, c);
        float x[16];
        widen_raw_row<DTYPE>(x, raw);
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = x[e] * sc[e];       // sign included: a sign commutes with every rounding below
        divide_by_norm(x, lds_read<float>(NORM_AT + 4 * (row - row0)));
        fwht_wave<B>(x, ls);
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = (x[e] * unit) * g[e >> 1];

        // ---------------- amplitude level and phase bin of the lane's 8 pairs
        float a2[8], most = 0.0f;
        unsigned ia[8], ip[8];                                  // times 4 and 8: byte offsets into the tables
        bool upper[8];                                          // angle in [pi, 2 pi)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float x0 = x[2 * k], x1 = x[2 * k + 1];
            a2[k] = __builtin_fmaf(x1, x1, x0 * x0);
            most = fmaxf(most, a2[k]);
            upper[k] = (x1 < 0.0f) || (x1 == 0.0f && x0 < 0.0f);
        }
        if (lut && __ballot(!(most <= PF_LUT_MAX_A2)) == 0ull) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int cell = (int)(__float_as_uint(a2[k]) >> 18) - (int)PF_AMP_BASE;
                ia[k] = lds_read<uint8_t>(AMP_AT + (uint32_t)min(max(cell, 0), PF_AMP_CELLS - 1));
                const float x0 = x[2 * k], x1 = x[2 * k + 1];
                const uint32_t at = polar_phase_cell(x0, x1, upper[k], [](float s) { return __builtin_amdgcn_rcpf(s); });
                ip[k] = 8u * lds_read<uint8_t>(PHASE_AT + at) + (upper[k] ? 4u * (unsigned)Np : 0u);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float t = lds_read<float>(THR_AT + 4 + ia[k]);
                const lds_f32x2_t b = lds_read<lds_f32x2_t>(DIR_AT + 8 + ip[k]);
                ia[k] = a2[k] > t ? ia[k] + 4u : ia[k];
                ip[k] = __builtin_fmaf(b[0], x[2 * k + 1], -(b[1] * x[2 * k])) >= 0.0f ? ip[k] + 8u : ip[k];
            }
        } else {
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
        }
        unsigned idx[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) idx[k] = ((ia[k] >> 2) << bits_p) + (a2[k] == 0.0f ? 0u : ip[k] >> 3);

        // ---------------- pack: the lane's 8 fields are exactly `bits` bytes, byte aligned in the row
        if (active) store_fields(packed + (int64_t)row * p.row_bytes, p.row_bytes, p.d_in, c, idx, p.bits);
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
    const unsigned blocks = (unsigned)((p.d_out + rows - 1) / rows);
    // Few rows of many slabs: several workgroups share a row, down to an item per wave, each with all slab sums of its own
    // (us by the trace at 5 + 6 bits, bf16, all options, one workgroup a row / so: 16 x 40960 23.4 / 12.1, 64 x 65536 36.0 / 22.1).
    int parts = 1;
    if (rows == 1) parts = std::max(1, std::min((n_slabs + PF_WAVES - 1) / PF_WAVES, 2 * PF_CUS / p.d_out));
    const size_t lds = PF_DIR_AT + 8 * ((size_t)(1 << bits_p) + 1);
    hipLaunchKernelGGL((k_encode_polar<DTYPE, B>), dim3(blocks, (unsigned)parts), dim3(PF_THREADS), lds, p.stream, W, ldw, p, levels, bits_a,
                       bits_p, norms_ready ? norms : nullptr, norms, packed, n_slabs, rows);
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
