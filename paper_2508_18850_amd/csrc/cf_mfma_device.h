// Small helpers for the matrix cores of gfx950 shared by the kernels that use v_mfma_f32_16x16x32_f16.
//
// Operand layout of one 16 x 16 x 32 step, lane = 16 g + c (g = 0..3, c = 0..15):
//   A: the lane holds A[i = c][k = 8 g .. 8 g + 7]      B: the lane holds B[k = 8 g .. 8 g + 7][j = c]
//   result: the lane holds D[i = 4 g + rr][j = c], rr = 0..3
#ifndef CF_MFMA_DEVICE_H
#define CF_MFMA_DEVICE_H

#include "cf_lanes_device.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cf {
namespace mfma {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma16(const h8 &a, const h8 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// w[u] = row u, eight adjacent columns  ->  f[c] = column c, rows 0..7 (8 x 8 transpose of 16-bit values in a lane):
// turns eight 16-byte pieces of row-major rows into eight B operands (contraction over the rows).
__device__ __forceinline__ void transpose8(const h8 *w, h8 (&f)[8])
{
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) {
        u32x4 e, o;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t lo = __builtin_bit_cast(u32x4, w[2 * d])[c2], hi = __builtin_bit_cast(u32x4, w[2 * d + 1])[c2];
            e[d] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);    // {lo.low half, hi.low half}
            o[d] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);    // {lo.high half, hi.high half}
        }
        f[2 * c2] = __builtin_bit_cast(h8, e);
        f[2 * c2 + 1] = __builtin_bit_cast(h8, o);
    }
}

// An fp32 operand of a matrix product that has to count in full: every row of the operand is scaled by a power of two that
// brings its largest value into [2^14, 2^15), and each value is cut into fp16 parts of eleven bits.  Three parts hold any
// fp32 value down to 2^-15 of the row's largest one exactly, below that to 2^-38 of the largest; two parts do the same for
// values of 22 bits, such as products of two fp16 values, down to 2^-17 of the largest.  Whatever the row's magnitude: a pair
// without the scale has an absolute step of 2^-24 (2e-3 of a value at 1e-5) and is NaN above 65504.  The scale is taken out
// where partial products are added.
template <int N>
struct Split {
    h8 part[N];
};
// largest magnitude of row c among this lane's values and those of the other contraction groups
__device__ __forceinline__ float row_max(float m) { return lanes::max_groups<16>(m); }
__device__ __forceinline__ float max_abs(const float (&v)[8], float m)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) m = fmaxf(m, fabsf(v[k]));
    return m;
}
// exponent of the scale of a row from its largest magnitude (at most 126: the inverse is a normal number)
__device__ __forceinline__ int scale_exp(float m) { return min(15 - (m <= 3.402823466e38f ? __builtin_amdgcn_frexp_expf(m) : 128), 126); }
template <int N>
__device__ __forceinline__ Split<N> split_scaled(const float (&v)[8], int e, float m)
{
    u32x4 p[N];
    float r[8], minus1 = -1.f;
    asm("" : "+s"(minus1));                                               // (kept a product: one v_fma_mix_f32 in place of a conversion and a difference)
#pragma unroll
    for (int k = 0; k < 8; ++k) r[k] = __builtin_amdgcn_ldexpf(v[k], e);
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
        for (int k = 0; k < 8; k += 2) {
            const auto t = __builtin_amdgcn_cvt_pkrtz(r[k], r[k + 1]);     // (cut off, not rounded: what is left keeps its sign)
            p[n][k / 2] = __builtin_bit_cast(uint32_t, t);
            r[k] = fmaf((float)t[0], minus1, r[k]);
            r[k + 1] = fmaf((float)t[1], minus1, r[k + 1]);
        }
    Split<N> s;
#pragma unroll
    for (int n = 0; n < N; ++n) s.part[n] = __builtin_bit_cast(h8, p[n]);
    if (__any(!(m <= 3.402823466e38f)))                                   // an infinity stays one, in the first part
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (!(fabsf(v[k]) <= 3.402823466e38f))
#pragma unroll
                for (int n = 1; n < N; ++n) s.part[n][k] = (_Float16)0.f;
    return s;
}

}  // namespace mfma
}  // namespace cf

#endif
