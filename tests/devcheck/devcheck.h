// Device functions of the library on the host: their header compiled by the host
// compiler, with stand-ins for the instructions it uses.  The reciprocal and
// reciprocal square root are estimates with a relative error of up to 2^-20, more
// than the hardware's, so that a result depends on the refinement that follows
// them and not on a lucky estimate.  A program that runs code of a whole wave
// defines the lane index and the ballot.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>

namespace dc {

// +-2^-20 at most, a fixed function of the argument's bits.
inline double wobble(double a) {
  uint64_t b;
  static_assert(sizeof(b) == sizeof(a));
  __builtin_memcpy(&b, &a, sizeof(a));
  b ^= b >> 31;
  b *= 0x9e3779b97f4a7c15ull;
  return (static_cast<double>(b >> 11) / static_cast<double>(1ull << 53) * 2.0 - 1.0) / 1048576.0;
}

[[noreturn]] inline void fail(const char* what) {
  std::printf("devcheck FAIL: %s\n", what);
  std::exit(1);
}

}  // namespace dc

inline double __builtin_amdgcn_rsq(double a) { return (1.0 + dc::wobble(a)) / std::sqrt(a); }
inline double __builtin_amdgcn_rcp(double a) { return (1.0 + dc::wobble(a)) / a; }
inline float __builtin_amdgcn_rcpf(float a) { return 1.0f / a; }
inline float __builtin_amdgcn_sqrtf(float a) { return std::sqrt(a); }

unsigned __lane_id();
unsigned long long __ballot(int predicate);

// kernels and their launches only have to parse
#undef __global__
#define __global__
#undef __launch_bounds__
#define __launch_bounds__(...)
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) ((void)0)
