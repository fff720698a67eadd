// Reductions between the lanes of a wavefront on the vector unit, without the LDS crossbar (a __shfl_xor is a
// ds_bpermute: some hundred cycles until its result is there, and the LDS pipe of the compute unit shared by all wavefronts).
//
// In the decode block, with shuffles / with these (us a layer, single launches, D = d_model): tiny shape 15.5 / 14.2; D 2056,
// 14 heads of 64, batch 3 22.9 / 20.2; Llama-2-7B shape 38.4 / 38.0; 64 heads of 64 over 8, D 2048, batch 1 28.8 / 23.0.
//
// A wavefront is seen as row groups of LPR = 8 or 16 consecutive lanes (the lanes that hold one row of a weight or
// cache tile); a value is reduced over the row groups, lane by lane.
#ifndef CF_LANES_DEVICE_H
#define CF_LANES_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cf {
namespace lanes {

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// lanes 32..63 of p <-> lanes 0..31 of q
__device__ __forceinline__ void swap32(float &p, float &q)
{
    const auto t = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, p), __builtin_bit_cast(unsigned, q), false, false);
    p = __builtin_bit_cast(float, (unsigned)t[0]);
    q = __builtin_bit_cast(float, (unsigned)t[1]);
}

// odd rows of 16 lanes of p <-> even rows of q
__device__ __forceinline__ void swap16(float &p, float &q)
{
    const auto t = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, p), __builtin_bit_cast(unsigned, q), false, false);
    p = __builtin_bit_cast(float, (unsigned)t[0]);
    q = __builtin_bit_cast(float, (unsigned)t[1]);
}

// v of lane i ^ 8 (a rotation by eight inside a row of 16)
__device__ __forceinline__ float xor8(float v) { return dpp_move<0x128>(v); }

// Sum / maximum over the row groups of a wavefront, in every lane.
template <int LPR>
__device__ __forceinline__ float sum_groups(float v)
{
    float p = v, q = v;
    swap32(p, q);
    v = p + q;
    p = v, q = v;
    swap16(p, q);
    v = p + q;
    return LPR == 8 ? v + xor8(v) : v;
}
template <int LPR>
__device__ __forceinline__ float max_groups(float v)
{
    float p = v, q = v;
    swap32(p, q);
    v = fmaxf(p, q);
    p = v, q = v;
    swap16(p, q);
    v = fmaxf(p, q);
    return LPR == 8 ? fmaxf(v, xor8(v)) : v;
}

// Sum / maximum over a row of 16 lanes, and over a half wavefront, in every lane of it.
__device__ __forceinline__ float sum_row(float v)
{
    v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);   // row_half_mirror: lane i <-> 7-i within 8 lanes
    return v + dpp_move<0x140>(v);   // row_mirror: lane i <-> 15-i within 16 lanes
}
__device__ __forceinline__ float max_row(float v)
{
    v = fmaxf(v, dpp_move<0xB1>(v));
    v = fmaxf(v, dpp_move<0x4E>(v));
    v = fmaxf(v, dpp_move<0x141>(v));
    return fmaxf(v, dpp_move<0x140>(v));
}
// v of this lane plus v of the lane 16 further in the same half wavefront (i ^ 16)
__device__ __forceinline__ float add16(float v)
{
    float p = v, q = v;
    swap16(p, q);
    return p + q;
}
__device__ __forceinline__ float sum_half(float v) { return add16(sum_row(v)); }
__device__ __forceinline__ float max_half(float v)
{
    float p = max_row(v), q = p;
    swap16(p, q);
    return fmaxf(p, q);
}

// Eight values per lane, each summed over the row groups, the sums dealt out: afterwards the lane of row group r holds
// those of values r * (LPR / 8) + j, j < LPR / 8.  A swap of halves between two values and an addition leave half as
// many values, so that it takes 12 (16 lanes per row) or 14 instructions where a sum in every lane takes 32 or 48.
template <int LPR>
__device__ __forceinline__ void fold8(const float (&v)[8], float (&out)[LPR / 8])
{
    static_assert(LPR == 8 || LPR == 16, "rows of 8 or 16 lanes");
    float h[4], t[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float p = v[j], q = v[j + 4];
        swap32(p, q);
        h[j] = p + q;                       // lanes 0..31: value j, lanes 32..63: value j + 4
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        float p = h[j], q = h[j + 2];
        swap16(p, q);
        t[j] = p + q;                       // odd rows of 16 lanes: two values further on
    }
    if constexpr (LPR == 16) {
        out[0] = t[0];
        out[1] = t[1];
    } else {
        const bool odd = (threadIdx.x & 8) != 0;      // keeps the second value, gives the first
        out[0] = (odd ? t[1] : t[0]) + xor8(odd ? t[0] : t[1]);
    }
}

}  // namespace lanes
}  // namespace cf

#endif
