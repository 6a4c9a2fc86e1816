// Standalone helix / intrusion angles of a given fibre field about an axis: a
// streaming map (12 bytes of e3 + 1 byte of mask in, 8 bytes of angles + 1 byte
// of flags out), bound by memory.  Voxels are taken by their flat index, so rows
// of any width fill the lanes and every access of a wave is contiguous; a lane
// takes 4 voxels and issues all their loads before the first is used.  VEC: the
// lane's voxels are neighbours, in 16-byte accesses; else they lie 64 apart.
// 250 x 510 x 509 with a mask takes 234 us (5.8 TB/s of required bytes, part of it
// from the Infinity Cache; a large copy reaches 4.7); one row per wave with 4
// neighbouring voxels a lane in 4-byte accesses, as before, took 468.
#include "st_device.h"

namespace st {
namespace {

constexpr int kPer = 4;             // voxels per lane
constexpr int kBlock = 256 * kPer;  // voxels per block

template <bool VEC>
__global__ __launch_bounds__(256) void k_angles(const AnglesParams p) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // voxel v of the lane is i0 + v * step
  constexpr int step = VEC ? 1 : 64;
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kBlock + wave * 64 * kPer + (VEC ? kPer * lane : lane);
  float e[3][kPer];
  uint8_t m[kPer];
#pragma unroll
  for (int v = 0; v < kPer; ++v) m[v] = 1;
  if constexpr (VEC) {  // n is a multiple of 4: a lane's voxels are all inside or all outside
    if (i0 >= p.n) return;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float4 t = *reinterpret_cast<const float4*>(p.e3 + c * p.n + i0);
      e[c][0] = t.x; e[c][1] = t.y; e[c][2] = t.z; e[c][3] = t.w;
    }
    if (p.mask != nullptr) {
      const uint32_t t = *reinterpret_cast<const uint32_t*>(p.mask + i0);
#pragma unroll
      for (int v = 0; v < kPer; ++v) m[v] = static_cast<uint8_t>(t >> (8 * v));
    }
  } else {
#pragma unroll
    for (int v = 0; v < kPer; ++v) {
      const int64_t i = i0 + v * step < p.n ? i0 + v * step : p.n - 1;
#pragma unroll
      for (int c = 0; c < 3; ++c) e[c][v] = p.e3[c * p.n + i];
      if (p.mask != nullptr) m[v] = p.mask[i];
    }
  }
  // (z, y, x) of a flat index in float64, exact below 2^51: (i + 1/2) / nx lies at
  // least 1 / (2 nx) from an integer, the product's rounding error below that
  const double dnx = static_cast<double>(p.nx), dny = static_cast<double>(p.ny);
  float ha[kPer], ia[kPer];
  uint32_t flag_word = 0;
#pragma unroll
  for (int v = 0; v < kPer; ++v) {
    ha[v] = 0.f;
    ia[v] = 0.f;
    uint32_t fl = ST_FLAG_OUTSIDE_MASK;
    if (m[v] != 0) {
      const double di = static_cast<double>(i0 + v * step);
      const double row = floor((di + 0.5) * p.inv_nx);
      const double px = fma(-row, dnx, di);
      const double pz = floor((row + 0.5) * p.inv_ny);
      const double py = fma(-pz, dny, row);
      fl = fibre_angles(e[0][v], e[1][v], e[2][v], p.center, p.dir, pz, py, px, ha[v], ia[v]) ? ST_FLAG_ON_AXIS : 0u;
    }
    flag_word |= fl << (8 * v);
  }
  if constexpr (VEC) {
    if (p.ha) *reinterpret_cast<float4*>(p.ha + i0) = make_float4(ha[0], ha[1], ha[2], ha[3]);
    if (p.ia) *reinterpret_cast<float4*>(p.ia + i0) = make_float4(ia[0], ia[1], ia[2], ia[3]);
    if (p.flags) *reinterpret_cast<uint32_t*>(p.flags + i0) = flag_word;
  } else {
#pragma unroll
    for (int v = 0; v < kPer; ++v) {
      const int64_t i = i0 + v * step;
      if (i >= p.n) break;
      if (p.ha) p.ha[i] = ha[v];
      if (p.ia) p.ia[i] = ia[v];
      if (p.flags) p.flags[i] = static_cast<uint8_t>(flag_word >> (8 * v));
    }
  }
}

}  // namespace

hipError_t launch_angles(const AnglesParams& q, hipStream_t stream) {
  AnglesParams p = q;
  p.inv_nx = 1.0 / static_cast<double>(p.nx);
  p.inv_ny = 1.0 / static_cast<double>(p.ny);
  const int64_t blocks = (p.n + kBlock - 1) / kBlock;
  if (p.n < 1 || p.n >= (int64_t(1) << 51) || blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (p.vec_ok)
    hipLaunchKernelGGL(k_angles<true>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL(k_angles<false>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace st
