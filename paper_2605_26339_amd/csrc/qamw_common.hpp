// Shared device helpers of libqamw's HIP kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qamw {

constexpr int WAVE = 64;

// Element load widened to fp32.  bf16 storage is the upper half of an fp32: widening is exact.
template <int DTYPE> struct Elem;
template <> struct Elem<0> {
    using type = float;
    static __device__ __forceinline__ float load(const void *base, int64_t i) {
        return reinterpret_cast<const float *>(base)[i];
    }
};
template <> struct Elem<1> {
    using type = uint16_t;
    static __device__ __forceinline__ float load(const void *base, int64_t i) {
        return __uint_as_float((uint32_t) reinterpret_cast<const uint16_t *>(base)[i] << 16);
    }
};

// Reciprocal with one Newton step: the correctly rounded quotient in all but a few rare cases
// (then one ulp off), at a third of the cost of the IEEE division sequence.
__device__ __forceinline__ float fast_recip(float s) {
    float q = __builtin_amdgcn_rcpf(s);
    float e = __builtin_fmaf(-s, q, 1.0f);
    return __builtin_fmaf(q, e, q);
}

// fp32 -> bf16 bits, round to nearest even (NaN stays a quiet NaN).
__device__ __forceinline__ uint32_t bf16_rne_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// One B-bit field of a little-endian bit stream held as dwords: field k sits at bit k*bits.
__device__ __forceinline__ uint32_t unpack_field(const uint32_t *row, int row_dwords, int k, int bits) {
    uint32_t bit = (uint32_t)k * (uint32_t)bits;
    uint32_t w = bit >> 5, sh = bit & 31u;
    uint64_t lo = row[w];
    uint64_t hi = (w + 1 < (uint32_t)row_dwords) ? row[w + 1] : 0u;
    return (uint32_t)(((hi << 32) | lo) >> sh) & ((1u << bits) - 1u);
}

// LDS by byte address.  In a kernel without statically sized LDS the dynamic block begins at 0: the constant part of an
// address then goes into the instruction's offset, where a pointer to the block costs an addition of 0 at every access.
template <typename T> __device__ __forceinline__ T lds_read(uint32_t at) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(at);
}
template <typename T> __device__ __forceinline__ void lds_write(uint32_t at, T v) {
    *reinterpret_cast<__attribute__((address_space(3))) T *>(at) = v;
}
__device__ __forceinline__ uint32_t lds_add(uint32_t at, uint32_t v) {   // returns what was there
    return __hip_atomic_fetch_add(reinterpret_cast<__attribute__((address_space(3))) uint32_t *>(at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
typedef float lds_f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t lds_u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t lds_u32x4_t __attribute__((ext_vector_type(4)));

// The value of the lane whose number differs in bit 0 or 1, and that of lane Q of the lane's group of four: one DPP move each
// (a shuffle through LDS takes some 120 cycles to come back).
template <int CTRL> __device__ __forceinline__ int dpp_move(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false); }
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) { return __int_as_float(dpp_move<CTRL>(__float_as_int(v))); }
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140, DPP_QUAD_REVERSE = 0x1B, DPP_ROW_ROTATE_8 = 0x128;
constexpr int dpp_quad_lane(int q) { return q * 0x55; }

// Sum over the 64 lanes of a wave in a fixed butterfly order (the same in every lane): lanes that differ in bit 0, then 1, ...
// The mirrors serve for bits 2 and 3, since the lanes of a group of four, then eight, hold the same by then.
__device__ __forceinline__ double wave_sum_of_16(double v) {     // each 16 lanes' sum
    auto step = [](double x, auto move) {
        return __hiloint2double(move(__double2hiint(x)), move(__double2loint(x)));
    };
    v += step(v, [](int w) { return dpp_move<DPP_XOR1>(w); });
    v += step(v, [](int w) { return dpp_move<DPP_XOR2>(w); });
    v += step(v, [](int w) { return dpp_move<DPP_HALF_MIRROR>(w); });
    v += step(v, [](int w) { return dpp_move<DPP_MIRROR>(w); });
    return v;
}
// a in the lanes 0-15 and 32-47, b in the others: each the sum of its value in a pair of neighbouring 16 lanes
__device__ __forceinline__ double wave_add_16(double a, double b) {
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// a in the lower half of the lanes, b in the upper half: each the sum of its values 32 lanes apart
__device__ __forceinline__ double wave_add_32(double a, double b) {
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = wave_sum_of_16(v);
    v = wave_add_16(v, v);
    return wave_add_32(v, v);
}
// wave_sum() of four values, to the bit: of v[r] in the lanes 16 r to 16 r + 15.
__device__ __forceinline__ double wave_sum_4(const double (&v)[4]) {
    const double a = wave_add_16(wave_sum_of_16(v[0]), wave_sum_of_16(v[1])), b = wave_add_16(wave_sum_of_16(v[2]), wave_sum_of_16(v[3]));
    return wave_add_32(a, b);
}

// The smallest of the 64 lanes' values, in every lane; no NaN among them.
__device__ __forceinline__ float wave_min(float v) {
    v = fminf(v, dpp_move<DPP_XOR1>(v));
    v = fminf(v, dpp_move<DPP_XOR2>(v));
    v = fminf(v, dpp_move<DPP_HALF_MIRROR>(v));
    v = fminf(v, dpp_move<DPP_MIRROR>(v));
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fminf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// The sum of the 64 lanes' values in a fixed order, the same in every lane.
__device__ __forceinline__ float wave_add(float v) {
    v += dpp_move<DPP_XOR1>(v);
    v += dpp_move<DPP_XOR2>(v);
    v += dpp_move<DPP_HALF_MIRROR>(v);
    v += dpp_move<DPP_MIRROR>(v);
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

}  // namespace qamw
