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

// 32-byte pack element: 8 time samples of one component of one site.
// Split precisions: 8 hi halves then 8 lo halves.  FP32: 8 floats.
struct alignas(16) Chunk {
    uint4 x, y;
};
// 48-byte pack element of the three-piece BF16 form: 8 hi, 8 mid, 8 lo.
struct alignas(16) Chunk3 {
    uint4 x, y, z;
};
template <int PREC>
using PackElem = typename std::conditional<PREC == SDC_PREC_BF16X3, Chunk3, Chunk>::type;

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
