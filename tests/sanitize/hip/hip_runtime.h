// What the lane code of the library's headers uses of HIP, for a build on the CPU.
#pragma once
#include <cstdint>
#define __device__
#define __host__
#define __constant__
#define __forceinline__ inline __attribute__((always_inline))
static inline int __popc(uint32_t x) { return __builtin_popcount(x); }
static inline int __ffs(uint32_t x) { return __builtin_ffs((int)x); }
static inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
static inline uint32_t __shfl_xor(uint32_t v, int) { return v; }
int __builtin_amdgcn_update_dpp(int, int, int, int, int, bool);  // of cross-lane code that no walk runs
