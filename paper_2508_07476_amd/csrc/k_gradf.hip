// Fused gradient pass: Gaussian-derivative gradient at scale sigma and the
// six-component outer product in one read of the input volume (filter
// arithmetic and products in float64, products stored as float32).
//
// Filter order per input plane: y (G and D), then x (three combinations), then
// z through per-column register windows, so that
//   g_z = Dz (Gx Gy V),  g_y = Gz (Gx Dy V),  g_x = Gz (Dx Gy V).
// A block of TY waves owns a TY (y) x 64 (x) tile of output columns and a chunk
// of z outputs (by default TY = 8 up to radius 6, where 8-row blocks still fit
// four waves per SIMD, else 4; a 4-row variant is also built up to radius 6 for
// the batch autotuner).  The input planes (z halo of R on each side, reflected at
// the faces) are taken in pairs.  For every pair the (TY + 2R) x (64 + 2R) input
// tiles are staged in LDS, in two buffers used by alternate pairs.  A pair's loads
// stay raw in registers (converted only when staged: a conversion beside the load
// waits for it) and have a whole pair's work to arrive: they are issued between
// the x and the z filter of the pair two before and staged at the same point of
// the next.  Each wave filters along y the 64 + 2R columns of its own tile row,
// which only it reads in the x filter, so one block barrier per pair (after the
// staging) suffices: a wave that writes pair j + 1's buffer has passed pair j's
// barrier, and one that would overwrite pair j's buffer (at j + 2) waits at pair
// j + 1's for every wave to finish reading it.
//
// What bounds the pass is VALU issue and LDS reads, each busy for about two thirds
// of it, at a clock held down by power.  The pairs save both: the y filter takes
// three wave steps for two planes instead of four (the 2R columns past the 64 of
// both planes fill one step together), and the x filter gives each half wave one
// plane, two neighbouring columns to a lane, so that a value read serves both (40 %
// fewer LDS bytes a voxel at R = 8; the sums return to their columns through LDS).
// Six-row tiles at radius 8 would stage less but leave room for one block a
// compute unit (8.6 ms below).  Times of the pass, u16: 512 x 1024 x 1024 at radius
// 8: 7.26 ms with the loads waited for where they were issued, 5.98 plane by plane,
// 5.32 by pairs; a masked 512^3 at radius 6: 1.28 ms plane by plane, 1.10 by pairs.
//
// Each column's z window lives in registers; the loop is expanded over the window's
// slots (a fold over an index sequence), so every plane's results land in a register
// fixed at compile time and the window never moves.
// Products leave with non-temporal stores into workspace planes whose rows have
// the workspace pitch (the input volume has rows of nx).
#include <utility>
#include "st_device.h"

namespace st {
namespace {

// Block `blk` of the gradient pass over the volume described by p (taps wg, wd).
// MASKED: only the runs of marked cells along z are computed (p.cells).
template <int R, typename Tin, int TY, bool MASKED = false>
__device__ __forceinline__ void grad_fused_block(const GradGeo& p, const Taps& wg, const Taps& wd, int64_t blk) {
  constexpr int W = 2 * R + 1;
  constexpr int TX = kGradTX;
  constexpr int NT = TX * TY;  // threads: one per output column of the tile
  constexpr int RX = TX + 2 * R, RY = TY + 2 * R;
  constexpr int NSTAGE = (RX * RY + NT - 1) / NT;  // staged elements per thread
  // The smoothing taps are symmetric about the centre (bit for bit, as built):
  // only taps 0..R are read, so R + 1 of them occupy scalar registers.
  auto tg = [&](int k) { return wg.w[k <= R ? k : 2 * R - k]; };
  constexpr int NP = 2;          // input planes per step (see above)
  constexpr int S = W + NP - 1;  // slots of a z window
  // doubles a wave keeps to itself: G and D of its row in each plane, filtered along
  // y, then (the x filter has read them) the three results of its 64 columns
  constexpr int NY = 2 * RX > 3 * TX ? 2 * NP * RX : 3 * NP * TX;
  __shared__ float raw[2][NP][RY * RX];  // input planes of a step (exact in float32), alternating
  __shared__ __attribute__((aligned(16))) double own[TY][NY];

  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * 64 + tx;
  // Blocks are dealt round-robin to the 8 XCDs (each with its own L2); give each
  // XCD a contiguous run of tiles so that tiles sharing halo rows meet in one L2.
  const int64_t nblk = p.x_tiles * p.y_tiles * p.nchunks;
  int64_t b = blk;
  if constexpr (MASKED) {
    // runs of four tile rows, dealt to the XCDs in turn: with one long run each, an
    // XCD at the edge of the mask would end early
    const int64_t run = 4 * p.x_tiles, whole = nblk / (8 * run) * (8 * run);
    if (b < whole) b = (b / 8 / run * 8 + b % 8) * run + b / 8 % run;
  } else if (nblk % 8 == 0) {
    b = (b % 8) * (nblk / 8) + b / 8;
  }
  const int64_t xt = b % p.x_tiles;
  b /= p.x_tiles;
  const int64_t yt = b % p.y_tiles;
  const int chunk_id = static_cast<int>(b / p.y_tiles);
  const int64_t x0 = xt * TX, y0 = yt * TY;
  const int64_t nz = p.nz, ny = p.ny, nx = p.nx;
  // z positions fit in 32 bits (each size < 2^31): their compares and the
  // reflection stay on the scalar unit; element offsets are 64-bit
  const int nzi = static_cast<int>(nz);
  const int c0 = chunk_id * static_cast<int>(p.chunk);
  const int clen = (nzi - c0) < p.chunk ? (nzi - c0) : static_cast<int>(p.chunk);
  const int64_t plane = ny * nx;  // < 2^31 (checked by the host)
  const Tin* vol = static_cast<const Tin*>(p.vol);

  // in-plane offsets of this thread's staging slots (reflected at the faces)
  int off[NSTAGE];
#pragma unroll
  for (int j = 0; j < NSTAGE; ++j) {
    int s = tid + NT * j;
    if (s >= RX * RY) s = RX * RY - 1;  // padding slots repeat the last element
    const int row = s / RX, col = s - (s / RX) * RX;
    const int gy = reflect_lane(static_cast<int>(y0) - R + row, static_cast<int>(ny));
    const int gx = reflect_lane(static_cast<int>(x0) - R + col, static_cast<int>(nx));
    off[j] = gy * static_cast<int>(nx) + gx;
  }
  auto run = [&](int z0, int len) {  // output planes z0 .. z0 + len - 1
    const int nplanes = len + 2 * R;  // at least 3
    const int nsteps = (nplanes + NP - 1) / NP;  // a last step may repeat its plane
    // the input planes in flight, as loaded: a conversion here would wait for them
    Tin pf[NP][NSTAGE];
    auto fetch = [&](int j) {  // loads of step j's planes into pf
#pragma unroll
      for (int e = 0; e < NP; ++e) {
        const int i = NP * j + e;
        const int zi = z0 - R + (e == 0 || i < nplanes ? i : nplanes - 1);
        const Tin* src = vol + static_cast<int64_t>(reflect_lane(zi, nzi)) * plane;
#pragma unroll
        for (int t = 0; t < NSTAGE; ++t) pf[e][t] = src[off[t]];  // halo re-read by neighbours: keep cached
      }
    };

    auto stage = [&](int j) {  // the fetched planes into step j's buffer
#pragma unroll
      for (int e = 0; e < NP; ++e) {
        float* rb = raw[j & 1][e];
#pragma unroll
        for (int t = 0; t < NSTAGE; ++t) {
          const int s = tid + NT * t;
          if (NT * (t + 1) <= RX * RY || s < RX * RY) rb[s] = static_cast<float>(pf[e][t]);
        }
      }
    };

    auto wave_fence = [] {  // orders the wave's own LDS accesses
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    double* const mine = own[ty];

    // Filter the planes of step j (staged) along y then x, which leaves the three
    // partial results of the wave's columns in each in `mine`.  Then stage step
    // j + 1, whose loads have been in flight since the step before, and issue those of
    // step j + 2: the wait for loads also waits for the products stored before them,
    // which by then had the two filters' time to leave.
    auto filter_step = [&](int j) {
      __syncthreads();
      // y filter of the wave's own row; only this wave reads it, so no block barrier
      // separates it from the x filter.  First 64 columns of each plane, then the 2 R
      // left of all planes together.
#pragma unroll
      for (int q = 0; q <= NP; ++q) {
        const int e = q < NP ? q : tx / (2 * R);
        const int col = q < NP ? tx : 64 + tx - 2 * R * e;
        if (q < NP || tx < 2 * R * NP) {
          const float* rb = raw[j & 1][e] + ty * RX + col;
          double g = 0.0, d = 0.0;
#pragma unroll
          for (int k = 0; k < W; ++k) {
            const double v = rb[k * RX];
            g = fma(tg(k), v, g);
            d = fma(wd.w[k], v, d);
          }
          mine[2 * e * RX + col] = g;
          mine[(2 * e + 1) * RX + col] = d;
        }
      }
      wave_fence();
      // x filter: 64 / NP lanes for each plane, NP neighbouring columns a lane (each
      // value read once for all of them)
      double ga[NP], gb[NP], dc[NP];
#pragma unroll
      for (int v = 0; v < NP; ++v) ga[v] = gb[v] = dc[v] = 0.0;
      const int e = tx / (64 / NP), c0 = NP * (tx % (64 / NP));
      const double* const us = mine + 2 * e * RX + c0;
#pragma unroll
      for (int i = 0; i < W + NP - 1; ++i) {
        const double u = us[i], w = us[RX + i];
#pragma unroll
        for (int v = 0; v < NP; ++v) {
          const int k = i - v;
          if (k < 0 || k >= W) continue;
          ga[v] = fma(tg(k), u, ga[v]);
          dc[v] = fma(wd.w[k], u, dc[v]);
          gb[v] = fma(tg(k), w, gb[v]);
        }
      }
      wave_fence();  // the sums are formed: their inputs' place is free
#pragma unroll
      for (int v = 0; v < NP; ++v) {
        double* const res = mine + TX * e + c0 + v;
        res[0] = ga[v];            // Gx Gy V -> Dz gives g_z
        res[NP * TX] = gb[v];      // Gx Dy V -> Gz gives g_y
        res[2 * NP * TX] = dc[v];  // Dx Gy V -> Gz gives g_x
      }
      wave_fence();
      if (j + 1 < nsteps) {
        stage(j + 1);
        if (j + 2 < nsteps) fetch(j + 2);
      }
    };

    const bool active = (x0 + tx < nx) && (y0 + ty < ny);
    const int64_t out_col = (y0 + ty) * p.opitch + (x0 + tx);
    const int64_t out_plane = ny * p.opitch;

    // z windows: slot j mod S holds the column's partial results of input plane j (W
    // of them are live).  The plane loop is expanded S times so that every slot index
    // is static (no register moves)
    double wa[S], wb[S], wc[S];
    fetch(0);
    stage(0);
    fetch(1);
#pragma unroll 1
    for (int jb = 0; jb < nplanes; jb += S) {  // block-uniform trip count
      auto step = [&]<int J>(std::integral_constant<int, J>) {  // planes jb + J .. jb + J + NP - 1
        if (jb + J < nplanes) {
          filter_step((jb + J) / NP);
#pragma unroll
          for (int e = 0; e < NP; ++e) {
            const int j = jb + J + e;
            wa[J + e] = mine[TX * e + tx];
            wb[J + e] = mine[TX * (NP + e) + tx];
            wc[J + e] = mine[TX * (2 * NP + e) + tx];
            if (j >= 2 * R && j < nplanes && active) {
              double gz = 0.0, gy = 0.0, gx = 0.0;
#pragma unroll
              for (int k = 0; k < W; ++k) {
                gz = fma(wd.w[k], wa[(J + e + k + NP) % S], gz);
                gy = fma(tg(k), wb[(J + e + k + NP) % S], gy);
                gx = fma(tg(k), wc[(J + e + k + NP) % S], gx);
              }
              const int64_t i = static_cast<int64_t>(z0 + j - 2 * R) * out_plane + out_col;
              __builtin_nontemporal_store(static_cast<float>(gz * gz), p.prod[0] + i);
              __builtin_nontemporal_store(static_cast<float>(gz * gy), p.prod[1] + i);
              __builtin_nontemporal_store(static_cast<float>(gz * gx), p.prod[2] + i);
              __builtin_nontemporal_store(static_cast<float>(gy * gy), p.prod[3] + i);
              __builtin_nontemporal_store(static_cast<float>(gy * gx), p.prod[4] + i);
              __builtin_nontemporal_store(static_cast<float>(gx * gx), p.prod[5] + i);
            }
          }
          wave_fence();  // the results are read: the next y filter overwrites them
        }
      };
      [&]<int... B>(std::integer_sequence<int, B...>) {
        (step(std::integral_constant<int, NP * B>{}), ...);
      }(std::make_integer_sequence<int, S / NP>{});
    }
  };
  if constexpr (MASKED) {
    const int64_t cxn = p.x_tiles, cyn = (ny + 7) / 8;  // cells are 64 columns wide, 8 rows high
    CellRuns runs(p.cells + y0 / 8 * cxn + xt, cyn * cxn, c0, clen);
    int ra, rlen;
#pragma unroll 1
    while (runs.next(ra, rlen)) {  // the same in every wave of the block
      run(ra, rlen);
      __syncthreads();  // the next run's first planes overwrite this one's last
    }
  } else {
    run(c0, clen);
  }
}

template <int R, typename Tin, int TY = grad_tile_rows(R)>
__global__ __launch_bounds__(64 * TY) __attribute__((amdgpu_waves_per_eu(TY == 8 || R <= 5 ? 4 : 3)))
void k_grad_fused(const GradFusedParams p) {
  grad_fused_block<R, Tin, TY>(p, p.wg, p.wd, blockIdx.x);
}

// With a wall mask that fills 0.49 of 512^3 u16 (sigma 1.5, rho 4) the gradient pass
// took 1.18 ms instead of 1.25 (plane by plane; every tile is resident at once, so the
// fullest column of blocks still ends it) and 0.04 for the cells, the integrations 1.10 and
// 1.02 instead of 1.38 and 1.35; 400 x 640 x 600 (sigma 2, rho 6): 1.56 instead of
// 2.01, 1.37 and 1.21 instead of 1.88 and 1.84.
template <int R, typename Tin, int TY = grad_tile_rows(R)>
__global__ __launch_bounds__(64 * TY) __attribute__((amdgpu_waves_per_eu(TY == 8 || R <= 5 ? 4 : 3)))
void k_grad_masked(const GradFusedParams p) {
  grad_fused_block<R, Tin, TY, true>(p, p.wg, p.wd, blockIdx.x);
}

// The mask by cells of 8^3 voxels: a thread per plane of a cell (eight rows of eight
// bytes, in flight together), a block for 32 neighbouring cells.
__global__ __launch_bounds__(256) void k_mask_cells(const uint8_t* mask, int64_t nz, int64_t ny, int64_t nx, int64_t cells,
                                                    uint8_t* out) {
  __shared__ int marked[32];
  const int k = threadIdx.x & 31, dz = threadIdx.x >> 5;
  const int64_t cy = (ny + 7) / 8, cx = (nx + 7) / 8;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 32 + k;
  if (threadIdx.x < 32) marked[k] = 0;
  __syncthreads();
  if (i < cells) {
    const int64_t x0 = i % cx * 8, y0 = i / cx % cy * 8, z = i / (cx * cy) * 8 + dz;
    uint64_t any = 0;
    if (z < nz) {
      uint64_t v[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const uint8_t* row = mask + (z * ny + (y0 + r < ny ? y0 + r : ny - 1)) * nx + x0;  // past the end: the last again
        if (x0 + 8 <= nx) {
          __builtin_memcpy(&v[r], row, 8);  // any alignment
        } else {
          v[r] = 0;
          for (int64_t x = x0; x < nx; ++x) v[r] |= row[x - x0];
        }
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) any |= v[r];
    }
    if (any != 0) marked[k] = 1;  // every writer writes the same
  }
  __syncthreads();
  if (threadIdx.x < 32 && i < cells) out[i] = static_cast<uint8_t>(marked[k]);
}

// Which cells of 8 x 8 x 64 voxels each pass has to compute (see MaskCells): the
// base cells within ceil(R / 8) cells along x, then y, then z.  Eight lanes share a
// cell, each taking every eighth of the rows around it.
__global__ __launch_bounds__(256) void k_needed_cells(MaskCells c, int64_t cz, int64_t cy, int64_t cx, int64_t xs) {
  const int part = threadIdx.x & 7;
  const int64_t j = static_cast<int64_t>(blockIdx.x) * 32 + (threadIdx.x >> 3);
  const int64_t i = j < cz * cy * xs ? j : cz * cy * xs - 1;
  const int64_t s = i % xs, y = i / xs % cy, z = i / (xs * cy);
  const int k = (c.reach + 7) / 8, side = 2 * k + 1;
  const int64_t xa = 8 * s - k > 0 ? 8 * s - k : 0, xb = 8 * s + 8 + k < cx ? 8 * s + 8 + k : cx;
  uint32_t need = 0;  // bit 0: y integration, 1: z integration, 2: products
  for (int r = part; r < side * side; r += 8) {
    const int dz = r / side - k, dy = r % side - k;
    if (z + dz < 0 || z + dz >= cz || y + dy < 0 || y + dy >= cy) continue;
    const uint8_t* row = c.base + ((z + dz) * cy + y + dy) * cx;
    uint32_t any = 0;
#pragma unroll 4
    for (int64_t x = xa; x < xb; ++x) any |= row[x];
    if (any != 0) need |= 4u | (dz == 0 ? 2u : 0u) | (dz == 0 && dy == 0 ? 1u : 0u);
  }
#pragma unroll
  for (int m = 1; m < 8; m *= 2) need |= __shfl_xor(need, m);
  if (part != 0 || j != i) return;
  c.y[i] = need & 1u;
  c.z[i] = need >> 1 & 1u;
  c.grad[i] = need >> 2;
}

hipError_t launch_mask_cells(const GradFusedParams& p, hipStream_t stream) {
  const MaskCells& c = p.mask;
  const int64_t cz = cells_of(p.nz), cy = cells_of(p.ny), cx = cells_of(p.nx), xs = p.x_tiles;
  const int64_t cells = cz * cy * cx;
  hipLaunchKernelGGL(k_mask_cells, dim3(static_cast<unsigned>((cells + 31) / 32)), dim3(256), 0, stream, c.mask, p.nz,
                     p.ny, p.nx, cells, c.base);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_needed_cells, dim3(static_cast<unsigned>((cz * cy * xs + 31) / 32)), dim3(256), 0, stream, c, cz,
                     cy, cx, xs);
  return hipGetLastError();
}

// One launch over a table of volumes.  Each entry's block range starts on a
// multiple of 8, so the XCD-aware remap inside a volume sees its own blocks
// dealt round-robin to the 8 XCDs as in a launch of its own.
template <int R, typename Tin, int TY>
__global__ __launch_bounds__(64 * TY) __attribute__((amdgpu_waves_per_eu(TY == 8 || R <= 5 ? 4 : 3)))
void k_grad_fused_grouped(const GradFusedGroup p) {
  const int64_t b = blockIdx.x;
  const int e = group_entry(p.g.first, p.g.count, b);
  const GradGeo g = p.g.geo[e];
  const int64_t local = b - p.g.first[e];
  if (local >= g.x_tiles * g.y_tiles * g.nchunks) return;  // alignment padding (block-uniform)
  grad_fused_block<R, Tin, TY>(g, p.wg, p.wd, local);
}

template <typename Tin, int R>
hipError_t launch_r(const GradFusedParams& p, hipStream_t stream) {
  const int64_t blocks = p.x_tiles * p.y_tiles * p.nchunks;
  if (p.cells != nullptr) {
    const hipError_t e = launch_mask_cells(p, stream);
    if (e != hipSuccess) return e;
    if (p.rows == grad_tile_rows(R)) {
      hipLaunchKernelGGL((k_grad_masked<R, Tin>), dim3(static_cast<unsigned>(blocks)), dim3(kGradTX, grad_tile_rows(R)),
                         0, stream, p);
      return hipGetLastError();
    }
    if constexpr (grad_rows_supported(R, 4) && grad_tile_rows(R) != 4) {
      if (p.rows == 4) {
        hipLaunchKernelGGL((k_grad_masked<R, Tin, 4>), dim3(static_cast<unsigned>(blocks)), dim3(kGradTX, 4), 0, stream,
                           p);
        return hipGetLastError();
      }
    }
    return hipErrorInvalidValue;
  }
  if (p.rows == grad_tile_rows(R)) {
    hipLaunchKernelGGL((k_grad_fused<R, Tin>), dim3(static_cast<unsigned>(blocks)), dim3(kGradTX, grad_tile_rows(R)),
                       0, stream, p);
    return hipGetLastError();
  }
  if constexpr (grad_rows_supported(R, 4) && grad_tile_rows(R) != 4) {
    if (p.rows == 4) {
      hipLaunchKernelGGL((k_grad_fused<R, Tin, 4>), dim3(static_cast<unsigned>(blocks)), dim3(kGradTX, 4), 0,
                         stream, p);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace

template <typename Tin, int R>
hipError_t launch_grouped_r(int rows, const GradFusedGroup& p, int64_t blocks, hipStream_t stream) {
  if (rows == grad_tile_rows(R)) {
    hipLaunchKernelGGL((k_grad_fused_grouped<R, Tin, grad_tile_rows(R)>), dim3(static_cast<unsigned>(blocks)),
                       dim3(kGradTX, grad_tile_rows(R)), 0, stream, p);
    return hipGetLastError();
  }
  if constexpr (grad_rows_supported(R, 4) && grad_tile_rows(R) != 4) {
    if (rows == 4) {
      hipLaunchKernelGGL((k_grad_fused_grouped<R, Tin, 4>), dim3(static_cast<unsigned>(blocks)), dim3(kGradTX, 4), 0,
                         stream, p);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

hipError_t launch_grad_fused(int R, int in_dtype, const GradFusedParams& p, hipStream_t stream) {
#define ST_CASE(r) case r: return in_dtype == ST_DTYPE_U16 ? launch_r<uint16_t, r>(p, stream) \
                                                           : launch_r<float, r>(p, stream);
  switch (R) { ST_CASE(1) ST_CASE(2) ST_CASE(3) ST_CASE(4) ST_CASE(5) ST_CASE(6) ST_CASE(7) ST_CASE(8)
    default: return hipErrorInvalidValue; }
#undef ST_CASE
}

hipError_t launch_grad_fused_grouped(int R, int in_dtype, int rows, const GradFusedGroup& p, int64_t blocks,
                                     hipStream_t stream) {
  if (blocks < 1) return hipSuccess;
#define ST_CASE(r) case r: return in_dtype == ST_DTYPE_U16 ? launch_grouped_r<uint16_t, r>(rows, p, blocks, stream) \
                                                           : launch_grouped_r<float, r>(rows, p, blocks, stream);
  switch (R) { ST_CASE(1) ST_CASE(2) ST_CASE(3) ST_CASE(4) ST_CASE(5) ST_CASE(6) ST_CASE(7) ST_CASE(8)
    default: return hipErrorInvalidValue; }
#undef ST_CASE
}

}  // namespace st
