// Device helpers the kernels share: 128-bit loads from a part of a read-only tensor, reciprocals.
#ifndef CF_STREAM_DEVICE_H
#define CF_STREAM_DEVICE_H

#include "cf_plan_arith.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cf {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));   // eight fp16 values = one 128-bit load

constexpr uint32_t kNoLoad = 0x80000000u;      // beyond the end of any part: for a lane with nothing to load
// Base and size are the same in all lanes; they are read from the first one, or the compiler, where it cannot see that, puts
// a loop over the lanes' values around every load.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>((uint64_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
// Part of a read-only tensor that is streamed once: raw buffer resource + 128-bit loads (AUX 2: non-temporal).  The buffer ends where
// the part ends (a slice of rows, a split of the cached rows; 0 bytes: nothing to load), so that a load past it costs no
// comparison: the hardware skips the access and returns zeros.  The whole offset is per lane, since the range check covers it
// then.  (A comparison and a select per load, and a wave-uniform offset beside them, were five instructions a load; a condition
// around a load is a branch, and the registers loaded on two paths are copied, behind a wait for the load, where the paths meet.)
template <int AUX>
struct Part {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Part(const void *base, uint32_t bytes) : r(buffer_of(base, bytes)) {}
    __device__ __forceinline__ h8 ld(uint32_t off) const { return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX)); }
};

// What fdiv takes for a divisor of this workgroup.
__device__ __forceinline__ float reciprocal(int d) { return __builtin_amdgcn_rcpf((float)d); }

}  // namespace cf

#endif
