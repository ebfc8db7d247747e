// Device types and helpers shared by the kernels of several files.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

#include "sdc_internal.h"

namespace sdc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Pack element: 8 time samples of one component of one site, in pieces of 16
// bytes.  Split precisions: 8 hi halves, then 8 lo halves.  FP32: 4 + 4 floats.
struct alignas(16) Chunk {
    uint4 x, y;
};
// Three-piece BF16 form: 8 hi, 8 mid, 8 lo.
struct alignas(16) Chunk3 {
    uint4 x, y, z;
};
template <int PREC>
using PackElem = typename std::conditional<PREC == SDC_PREC_BF16X3, Chunk3, Chunk>::type;

// The packs of the two-piece splits hold a plane of hi and a plane of lo
// halves: the pass over the hi halves alone then fetches no lo halves in its
// cache lines.  The other forms multiply all pieces of an element at once and
// keep them side by side.  Fused ms side by side / in planes (origins x lags):
// BF16 sc 36^3 128 x 256 1028 / 1018, sc 30^3 100 x 100 122.3 / 119.0, ball of
// 20 011 points 64 x 128 53.1 / 52.6; FP32 sc 21x20x19 50 x 100 20.9 / 21.3,
// BF16x3 90x90 50 x 64 8.10 / 8.20.
__host__ __device__ constexpr bool pack_planes(int prec) {
    return prec == SDC_PREC_SPLIT_BF16 || prec == SDC_PREC_SPLIT_FP16;
}
// What a pack's index counts: pieces of a plane, or elements.
template <int PREC>
using PackUnit = typename std::conditional<pack_planes(PREC), uint4, PackElem<PREC>>::type;
// Pieces per plane of the A and the B pack.
template <class Args>
__device__ __forceinline__ int64_t pack_plane_a(const Args& a) {
    return ((int64_t)3 * a.O8 + 1) * a.n_pad;
}
template <class Args>
__device__ __forceinline__ int64_t pack_plane_b(const Args& a) {
    return (int64_t)a.n_phase * 3 * a.F8 * a.n_pad;
}

__device__ inline uint32_t bf16_bits(float v) {
    __bf16 b = (__bf16)v;  // round to nearest even
    return (uint32_t)__builtin_bit_cast(uint16_t, b);
}
__device__ inline uint32_t f16_bits(float v) {
    _Float16 b = (_Float16)v;
    return (uint32_t)__builtin_bit_cast(uint16_t, b);
}
__device__ inline float bf16_val(uint32_t bits) {
    return (float)__builtin_bit_cast(__bf16, (uint16_t)bits);
}
__device__ inline float f16_val(uint32_t bits) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}

// Fixed-point image of v (deterministic mode), rounded to nearest.
__device__ inline unsigned long long to_fixed(double v) {
    return (unsigned long long)__double2ll_rn(v * kFixedScale);
}

__device__ inline int pmod_dev(int a, int m) {
    int r = a % m;
    return r < 0 ? r + m : r;
}

}  // namespace sdc
