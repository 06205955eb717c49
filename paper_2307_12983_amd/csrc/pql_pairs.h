// fp32 values as scaled fp16 pairs, for kernels that multiply on the fp16 matrix cores at 32-bit precision
// (pql_split.hip, the weight-gradient kernel of pql_gemm.hip).  Device code only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pql {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Power-of-two scale that brings a largest magnitude m to [2^14, 2^15), and its inverse.  The exponent is clamped so that both
// are normal numbers (zero rows, subnormals, infinities).
__device__ __forceinline__ float scale_for(float m, float& inv) {
    int e = (int)(__float_as_uint(m) >> 23);
    e = e < 20 ? 20 : (e > 254 ? 254 : e);
    inv = __uint_as_float((unsigned)(e - 14) << 23);
    return __uint_as_float((unsigned)(254 + 14 - e) << 23);
}

// x s = hi + lo / 2^11, two values packed.  The factor keeps lo a normal number down to hi = 2^-14; lo products need sums of
// their own.  (The empty asm keeps the compiler from converting once for the pair and once more for the difference: hi is
// formed packed and read back by the fused multiply-add.)
constexpr float PAIR_LO = 2048.f;
__device__ __forceinline__ void split16x2(float x0, float x1, float s, unsigned& hi, unsigned& lo) {
    const float y0 = x0 * s, y1 = x1 * s;
    const f16x2 a = {(_Float16)y0, (_Float16)y1};
    hi = __builtin_bit_cast(unsigned, a);
    asm("" : "+v"(hi));
    const f16x2 h = __builtin_bit_cast(f16x2, hi);
    const f16x2 l = {(_Float16)__fmaf_rn((float)h[0], -PAIR_LO, y0 * PAIR_LO), (_Float16)__fmaf_rn((float)h[1], -PAIR_LO, y1 * PAIR_LO)};
    lo = __builtin_bit_cast(unsigned, l);
}
__device__ __forceinline__ void split16(float x, float s, _Float16& hi, _Float16& lo) {
    const float y = x * s;
    hi = (_Float16)y;
    lo = (_Float16)((y - (float)hi) * PAIR_LO);
}

}  // namespace pql
