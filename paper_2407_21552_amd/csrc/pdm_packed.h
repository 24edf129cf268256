// pdm_packed.h -- device helpers on packed bytes, shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pdm {


typedef unsigned short us2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_min16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2, a),
                                                                  __builtin_bit_cast(us2, b)));
}
__device__ __forceinline__ uint32_t pk_max16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a),
                                                                  __builtin_bit_cast(us2, b)));
}
__device__ __forceinline__ uint32_t pk_add16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(us2, a) + __builtin_bit_cast(us2, b));
}
// difference, 0 where b > a
__device__ __forceinline__ uint32_t pk_sub_sat16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(us2, a),
                                                                      __builtin_bit_cast(us2, b)));
}
// bytes 0 and 2 of w in the two 16-bit halves
__device__ __forceinline__ uint32_t even_bytes(uint32_t w) { return w & 0x00FF00FFu; }
// bytes 1 and 3 of w in the two 16-bit halves
__device__ __forceinline__ uint32_t odd_bytes(uint32_t w) {
    return __builtin_amdgcn_perm(0u, w, 0x0c030c01u);
}
__device__ __forceinline__ uint32_t lo16(uint32_t w) { return w & 0xFFFFu; }
__device__ __forceinline__ uint32_t hi16(uint32_t w) { return w >> 16; }
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }

// Pointers typed in the global address space.  Kernel arguments are known to
// be global; pointers read from a descriptor are not, and would compile to
// flat accesses, which also count against the LDS wait counter and so stall
// the LDS-paced loops.
#define PDM_GLB __attribute__((address_space(1)))

// Work-groups are handed to the 8 XCDs round-robin (work-group b runs on XCD
// b % 8).  xcd_item maps work-group b to a work item so that runs of kXcdRun
// consecutive items land on one XCD at about the same time: neighbouring
// 64-line tiles of a row share 128-byte cache lines, and under one L2 the
// second tile finds the line the first one fetched.  The grid is rounded up
// to a multiple of kXcds * kXcdRun; work-groups past the last item return.
constexpr int kXcds = 8;
constexpr int kXcdRun = 4;
constexpr int64_t kXcdSpan = (int64_t)kXcds * kXcdRun;

__device__ __forceinline__ int64_t xcd_item(int64_t b) {
    const int64_t r = b % kXcdSpan;
    return (b - r) + (r % kXcds) * kXcdRun + r / kXcds;
}

}  // namespace pdm
