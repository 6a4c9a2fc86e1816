// Per-tile fallback of the surrogate to the structure-tensor path: flag the
// tiles that hold low-confidence voxels, gather each flagged tile with the
// path's halo into a crop stack, and write the crops' path outputs back over
// the surrogate's where the confidence is low.  All three kernels are plain
// copies and compares, bound by HBM.
#include "st_device.h"
#include "st_surrogate.h"

namespace st {
namespace {

constexpr int kRowThreads = 128;  // threads per crop row (gather, merge)

// Clears the flags of edges 64 and 128.
__global__ __launch_bounds__(256) void k_sg_clear_flags(const SgTileFlagParams p) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
#pragma unroll
  for (int k = 1; k < kSgTileEdges; ++k) {
    if (i >= 0 && i < p.tiles[k]) p.flags[k][i] = 0;
    i -= p.tiles[k];
  }
}

// One block per tile of edge 32 (a thread per column of 32 planes): it alone writes
// the tile's flag, and raises those of the tiles of edge 64 and 128 around it.
// Reads bound it: 192 x 256 x 250 takes 37 us; a wave per 64-voxel row segment, all
// raising the flags of all three grids, took 217.
constexpr int kFlagEdge = 32;
__global__ __launch_bounds__(kFlagEdge * kFlagEdge) void k_sg_tile_flags(const SgTileFlagParams p) {
  const int64_t tyn = (p.ny + kFlagEdge - 1) / kFlagEdge, txn = (p.nx + kFlagEdge - 1) / kFlagEdge;
  const int64_t t = blockIdx.x, tx = t % txn, ty = t / txn % tyn, tz = t / txn / tyn;
  const int64_t x = tx * kFlagEdge + threadIdx.x % kFlagEdge, y = ty * kFlagEdge + threadIdx.x / kFlagEdge;
  bool low = false;
  if (x < p.nx && y < p.ny) {
    const int64_t z0 = tz * kFlagEdge, plane = p.ny * p.nx, col = y * p.nx + x;
    constexpr int BATCH = 8;  // planes whose loads are in flight together
    for (int64_t z = z0; z < z0 + kFlagEdge && z < p.nz; z += BATCH) {
      float conf[BATCH];
      uint8_t inside[BATCH];
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const int64_t i = (z + k < p.nz ? z + k : p.nz - 1) * plane + col;  // past the end: the last again
        conf[k] = p.conf[i];
        inside[k] = p.mask == nullptr ? 1 : p.mask[i];
      }
#pragma unroll
      for (int k = 0; k < BATCH; ++k) low |= inside[k] != 0 && conf[k] < p.threshold;
    }
  }
  const int any = __syncthreads_or(low);
  if (threadIdx.x >= kSgTileEdges) return;
  const int k = static_cast<int>(threadIdx.x), s = 5 + k;
  if (k == 0) {
    p.flags[0][t] = any;
  } else if (any) {
    const int64_t kyn = (p.ny + (int64_t(1) << s) - 1) >> s, kxn = (p.nx + (int64_t(1) << s) - 1) >> s;
    __hip_atomic_store(p.flags[k] + ((tz >> k) * kyn + (ty >> k)) * kxn + (tx >> k), 1, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <class T>
__global__ __launch_bounds__(kRowThreads) void k_sg_gather(const SgGatherParams p) {
  const int64_t r = blockIdx.x;
  const int c = group_entry(p.first, p.count, r);
  const SgBox bx = p.boxes[c];
  const int64_t lr = r - p.first[c];
  const int64_t zz = lr / bx.cy, yy = lr - zz * bx.cy;
  const int64_t src = ((bx.z0 + zz) * p.ny + (bx.y0 + yy)) * p.nx + bx.x0;
  const int64_t dst = bx.off + lr * bx.cx;
  const T* in = static_cast<const T*>(p.vol);
  T* out = static_cast<T*>(p.cvol);
  for (int64_t x = threadIdx.x; x < bx.cx; x += kRowThreads) {
    out[dst + x] = in[src + x];
    if (p.mask != nullptr) p.cmask[dst + x] = p.mask[src + x];
  }
}

__global__ __launch_bounds__(kRowThreads) void k_sg_tile_merge(const SgTileMergeParams p) {
  const int64_t r = blockIdx.x;
  const int c = group_entry(p.first, p.count, r);
  const SgBox bx = p.boxes[c];
  const int64_t lr = r - p.first[c];
  const int64_t th = bx.ty1 - bx.ty0;
  const int64_t zz = bx.tz0 + lr / th, yy = bx.ty0 + lr % th;
  const int64_t cv = bx.cz * bx.cy * bx.cx;
  const int64_t crow = ((zz - bx.z0) * bx.cy + (yy - bx.y0)) * bx.cx - bx.x0;  // + x: index in the crop
  const int64_t vrow = (zz * p.ny + yy) * p.nx;
  for (int64_t x = bx.tx0 + threadIdx.x; x < bx.tx1; x += kRowThreads) {
    const int64_t i = vrow + x;
    if (p.mask != nullptr && p.mask[i] == 0) continue;
    if (!(p.conf[i] < p.threshold)) continue;
    const int64_t j = crow + x;
    if (p.e3) {
      p.e3[i] = p.pe3[3 * bx.off + j];
      p.e3[p.n + i] = p.pe3[3 * bx.off + cv + j];
      p.e3[2 * p.n + i] = p.pe3[3 * bx.off + 2 * cv + j];
    }
    if (p.fa) p.fa[i] = p.pfa[bx.off + j];
    if (p.ha) p.ha[i] = p.pha[bx.off + j];
    if (p.ia) p.ia[i] = p.pia[bx.off + j];
  }
}

bool fits_grid(int64_t blocks) { return blocks >= 1 && blocks <= 0x7fffffff; }

}  // namespace

hipError_t launch_sg_tile_flags(const SgTileFlagParams& p, hipStream_t stream) {
  int64_t tiles = 0;
  for (int k = 1; k < kSgTileEdges; ++k) tiles += p.tiles[k];
  if (!fits_grid((tiles + 255) / 256) || !fits_grid(p.tiles[0])) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_sg_clear_flags, dim3(static_cast<unsigned>((tiles + 255) / 256)), dim3(256), 0, stream, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sg_tile_flags, dim3(static_cast<unsigned>(p.tiles[0])), dim3(kFlagEdge * kFlagEdge), 0, stream,
                     p);
  return hipGetLastError();
}

hipError_t launch_sg_gather(int dtype, const SgGatherParams& p, hipStream_t stream) {
  if (!fits_grid(p.rows) || p.count < 1) return hipErrorInvalidValue;
  if (dtype == ST_DTYPE_U16)
    hipLaunchKernelGGL(k_sg_gather<uint16_t>, dim3(static_cast<unsigned>(p.rows)), dim3(kRowThreads), 0, stream, p);
  else
    hipLaunchKernelGGL(k_sg_gather<float>, dim3(static_cast<unsigned>(p.rows)), dim3(kRowThreads), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_sg_tile_merge(const SgTileMergeParams& p, hipStream_t stream) {
  if (!fits_grid(p.rows) || p.count < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_sg_tile_merge, dim3(static_cast<unsigned>(p.rows)), dim3(kRowThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace st
