// The polar encoder's lookup tables: who makes them, and which cell a pair falls into.  Plain C++, so that it runs on the CPU too.
#pragma once
#include <cstdint>

namespace qamw {

// Lookup tables in place of the two binary searches, for workgroups that encode at least PF_LUT_ITEMS (row, slab) items (making
// them takes a workgroup 1 us).  Amplitude: by exponent and five mantissa bits of |x|^2, 16 octaves from 2^-10 on.  Phase: by
// x0 / (|x0| + |x1|), which falls with the angle in [0, pi), in 256 cells; its slope is at least half of the angle's, so with up
// to 256 bins no cell holds two boundaries.  An entry holds the code at the cell's beginning and the one boundary that may lie in it,
// which is tested as the searches test it.
constexpr int PF_LUT_ITEMS = 16;
constexpr int PF_AMP_CELLS = 512, PF_PHASE_CELLS = 256, PF_LUT_MIN_BINS = 8, PF_LUT_MAX_BINS = 256;
constexpr float PF_LUT_MAX_A2 = 1e30f;  // beyond, 1 / (|x0| + |x1|) is on its way to the subnormals: the searches

// What workgroup `part` of `parts` that share n_items encodes, and whether with tables for Np bins.
struct PolarPart {
    int from, to;
    bool tables;
};
constexpr PolarPart polar_part(int n_items, int part, int parts, int Np) {
    const int from = n_items * part / parts, to = n_items * (part + 1) / parts;
    return {from, to, to - from >= PF_LUT_ITEMS && Np >= PF_LUT_MIN_BINS && Np <= PF_LUT_MAX_BINS};
}

// The phase cell of a pair with |x|^2 <= PF_LUT_MAX_A2, its angle in [pi, 2 pi) taken less pi; recip: 1 / s to some units.
// The sum is kept at a normal number, so that the product is one between -1 and 1: of zeros and subnormals the reciprocal is
// infinite.  (Their |x|^2 is 0, and the phase of that is 0 whatever the cell.)
template <class Recip> constexpr uint32_t polar_phase_cell(float x0, float x1, bool upper, Recip recip) {
    const float place = (upper ? -x0 : x0) * recip(__builtin_fmaxf(__builtin_fabsf(x0) + __builtin_fabsf(x1), 0x1p-126f));
    const uint32_t at = (uint32_t)__builtin_fmaf(place, 0.5f * PF_PHASE_CELLS, 0.5f * PF_PHASE_CELLS);
    return at < (uint32_t)PF_PHASE_CELLS ? at : (uint32_t)PF_PHASE_CELLS - 1u;
}

}  // namespace qamw
