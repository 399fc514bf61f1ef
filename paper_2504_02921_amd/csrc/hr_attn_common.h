// Device pieces that the attention kernels share: fp8 expansion, row reductions, the sub-tile's page geometry.
#pragma once

#include <hip/hip_runtime.h>

#include "hr_device_types.h"
#include "hr_layout.h"

namespace hr {

typedef __attribute__((ext_vector_type(8))) _Float16 halfx8;
typedef __attribute__((ext_vector_type(4))) _Float16 halfx4;
typedef __attribute__((ext_vector_type(2))) _Float16 halfx2;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(2))) float floatx2;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

constexpr float kLazyMax = 8.0f;     // by how much (log2 units) scores must exceed the running maximum before it follows

// 8 consecutive fp8 codes (one 64-bit LDS word) -> 8 halves, times a power of two.
// An E4M3 code s.eeee.mmm placed at bits 15, 13..7 of a half (sign kept, exponent and mantissa fields shifted down
// by one) reads as (-1)^s 2^(e-15) (1 + m/8), or (-1)^s 2^-14 (m/8) when e = 0: in both cases the E4M3 value
// (bias 7, subnormals m/8 * 2^-6) divided by 2^8.  So the conversion is a byte shuffle, two masks, a shift and one
// packed half multiplication by 2^8 * 2^k, exact while the product is a half.  (The hardware's scaled conversion
// instruction gives the same values but measured ~88 cycles per wavefront instruction, against 4 for these.)
// The two NaN codes (0x7f, 0xff) read as +-480; a pool never holds them.
__device__ __forceinline__ halfx8 fp8x8_to_half(uint2 w, halfx2 pow2) {
    auto pair = [&](unsigned x, unsigned sel) {
        const unsigned t = __builtin_amdgcn_perm(x, 0u, sel);                    // code bytes to the high byte of each 16-bit half
        const unsigned h = (t & 0x80008000u) | ((t & 0x7F007F00u) >> 1);
        halfx2 v;
        __builtin_memcpy(&v, &h, 4);
        return v * pow2;
    };
    const halfx2 a = pair(w.x, 0x050c040cu), b = pair(w.x, 0x070c060cu), c = pair(w.y, 0x050c040cu), d = pair(w.y, 0x070c060cu);
    halfx8 r;
    r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1]; r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
    return r;
}

// Reductions over lanes l and l ^ 32 (the two lanes that share a query row) through the VALU lane-swap instruction instead of an
// LDS round trip: v_permlane32_swap exchanges the upper half of its first operand with the lower half of its second, so
// with the same value in both the first result holds lanes 0..31 twice and the second lanes 32..63 twice.
__device__ __forceinline__ float row_max2(float x) {       // max over the two lanes of a row, in both
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row_sum2(float x) {       // sum over the two lanes of a row, in both (same bits in both)
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 2^8 times the power of two of a positive scale, as a pair of halves (clamped to the normal range of half)
__device__ __forceinline__ halfx2 fp8_expand_factor(float scale) {
    int e = (int)((__float_as_uint(scale) >> 23) & 0xFFu) - 127 + 8;
    e = e < -14 ? -14 : (e > 15 ? 15 : e);
    const _Float16 f = (_Float16)__uint_as_float((unsigned)(e + 127) << 23);
    return halfx2{f, f};
}

// The mantissa of a positive V scale, in [1, 2): what the expansion's power of two leaves for the probabilities
__device__ __forceinline__ float fp8_scale_mantissa(float scale) { return __uint_as_float((__float_as_uint(scale) & 0x007FFFFFu) | 0x3F800000u); }

}  // namespace hr
