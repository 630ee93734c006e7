// Device helpers that several kernel files share.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace atalib {

typedef __amdgpu_buffer_rsrc_t rsrc_t;

// Index of element (r, q) in a packed lower triangle.
__device__ __forceinline__ int64_t pidx(int64_t r, int64_t q) { return r * (r + 1) / 2 + q; }

template <typename OUT>
__device__ __forceinline__ void store_c(OUT* p, int beta, double v) {
    *p = beta ? (OUT)((double)*p + v) : (OUT)v;
}

// One 16-byte-per-lane copy into LDS.  A device function of its own: the host
// pass does not know the 16-byte form and would drop a kernel that holds it.
__device__ __forceinline__ void lds_copy16(rsrc_t r, void* lds, uint32_t voff, int soff = 0) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff, soff, 0, 0);
}

// Value of v in lane src (uniform) for every lane, through scalar registers.
__device__ __forceinline__ double lane_bcast(double v, int src) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, src);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), src);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float lane_bcast(float v, int src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
}

// Orders the LDS accesses of one wave (they complete in order; this keeps the
// compiler from moving them).
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

}  // namespace atalib
