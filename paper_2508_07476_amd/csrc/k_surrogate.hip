// Learned orientation surrogate: a dense 3-D CNN (five 3x3x3 convolutions with
// 32 channels and ReLU, a 1x1x1 head with 5 outputs) evaluated on the bf16
// matrix cores, float32 accumulation.
//
// Activations are channel-last bf16 ([voxel][32], 64 bytes per voxel).  A
// convolution is an implicit GEMM per tap: out[co][voxel] += W[co][ci] * in[ci][voxel
// + tap] with M = output channel (two 16-blocks), N = 16 consecutive voxels
// along x, K = the 32 input channels of one tap, one v_mfma_f32_16x16x32_bf16
// per (tap, M-block, N-block).  Operand layout of that instruction on gfx950
// (probed): lane l holds A[l % 16][8 (l / 16) + i] and B[8 (l / 16) + i][l % 16],
// i = 0..7, and receives D[4 (l / 16) + r][l % 16], r = 0..3 -- so each lane
// ends with 4 consecutive output channels of one voxel, an 8-byte channel-last
// store.
//
// Two kernels.  The first layer (k_sg_conv): a block of 8 waves owns 8 (y) x 32
// (x) output voxels and marches through a chunk of z planes; its weights (32 x 32
// bf16) and a ring of 3 input planes of 10 x 34 voxels (faces clamped) live in
// LDS.  The 32 -> 32 layers (k_sg_conv_ws, below: inference and training) keep
// their weights in registers.  Both issue the next plane's loads before the
// current plane's matrix products, and both take z chunks by sg_zchunk.
// The last layer's epilogue evaluates the head, the normalisation, FA,
// confidence, the mask and the helix / intrusion angles.
#include <algorithm>
#include <utility>

#include "st_device.h"
#include "st_surrogate.h"

namespace st {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int C = kSgChannels;
constexpr int TY = 8, TX = 32, RY = TY + 2, RX = TX + 2;
constexpr int NT = 64 * TY;         // threads per block: one wave per output row
constexpr int PLANE_VOX = RY * RX;  // voxels of one staged plane

__device__ __forceinline__ int64_t clampi(int64_t v, int64_t n) { return v < 0 ? 0 : (v >= n ? n - 1 : v); }

// Packs the float32 blob into bf16 operand layouts: layer 1 as [co][k] (k < 27 a
// tap, the rest 0), layers 2..5 as [tap][co][ci].
__global__ void k_sg_pack(const float* blob, __bf16* w1, __bf16* w25) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < C * 32) {
    const int co = static_cast<int>(i / 32), k = static_cast<int>(i % 32);
    w1[i] = static_cast<__bf16>(k < 27 ? blob[kSgOffW1 + co * 27 + k] : 0.f);
  }
  const int64_t per = 27 * C * C;
  if (i < 4 * per) {
    const int layer = static_cast<int>(i / per);  // 0 -> network layer 2
    const int64_t r = i % per;
    const int tap = static_cast<int>(r / (C * C)), co = static_cast<int>((r / C) % C),
              ci = static_cast<int>(r % C);
    w25[i] = static_cast<__bf16>(blob[kSgOffW2 + layer * kSgLayerStride + (co * C + ci) * 27 + tap]);
  }
}

// Outputs of one voxel from its five head values o = bh + Wh x5: unit fibre
// vector with the canonical sign, FA and confidence (sigmoids), the helix and
// intrusion angles; zeros outside the mask.
__device__ __forceinline__ void head_outputs(const SgConvParams& p, const float o[5], bool inside, int64_t z,
                                             int64_t yo, int64_t xv) {
  const int64_t vox = (z * p.ny + yo) * p.nx + xv;
  float ez = 0.f, ey = 0.f, ex = 0.f, fa = 0.f, conf = 0.f, ha = 0.f, ia = 0.f;
  if (inside) {
    const float nn = o[0] * o[0] + o[1] * o[1] + o[2] * o[2];
    if (nn > 0.f) {
      const float inv = 1.f / sqrtf(nn);
      ez = o[0] * inv; ey = o[1] * inv; ex = o[2] * inv;
    } else {
      ez = 1.f;
    }
    const float az = fabsf(ez), ay = fabsf(ey), ax = fabsf(ex);
    const float lead = (az >= ay && az >= ax) ? ez : (ay >= ax ? ey : ex);
    if (lead < 0.f) { ez = -ez; ey = -ey; ex = -ex; }
    fa = 1.f / (1.f + expf(-o[3]));
    conf = 1.f / (1.f + expf(-o[4]));
    if (p.has_axis)
      (void)fibre_angles(ez, ey, ex, p.center, p.dir, static_cast<double>(z), static_cast<double>(yo),
                         static_cast<double>(xv), ha, ia);
  }
  const int64_t nvox = p.n;
  if (p.e3) { p.e3[vox] = ez; p.e3[nvox + vox] = ey; p.e3[2 * nvox + vox] = ex; }
  if (p.fa) p.fa[vox] = fa;
  if (p.conf) p.conf[vox] = conf;
  if (p.ha) p.ha[vox] = ha;
  if (p.ia) p.ia[vox] = ia;
}

// Rounds of blocks that a launch over `tiles` x-y tiles of `planes` planes takes in z
// chunks of c, with per_cu blocks on a CU.
int64_t sg_rounds(int64_t tiles, int64_t planes, int64_t per_cu, int64_t c) {
  const int64_t cap = 256 * per_cu, blocks = tiles * ((planes + c - 1) / c);
  return (blocks + cap - 1) / cap;
}

// z planes per block.  A block pays about kChunkHead planes' time before its first
// output (the ring's first planes, the weights), so the launch takes about its rounds
// times (chunk + head): the chunk that makes this least, the largest such up to
// `most`.  A fixed 16 left a 48^3 volume's layers with 18 blocks: 83 us a layer,
// against 18.  masked: an unknown part of the blocks has work and the rest ends at
// once, so the chunk is the best for a half, three quarters and all of them together.
constexpr int64_t kChunkHead = 3;
int64_t sg_zchunk(int64_t tiles, int64_t planes, int64_t per_cu, int64_t most, bool masked) {
  const int64_t cap = 256 * per_cu;
  int64_t best = 1, cost = INT64_MAX;
  for (int64_t c = 1; c <= std::min(planes, most); ++c) {
    const int64_t blocks = tiles * ((planes + c - 1) / c);
    int64_t rounds = sg_rounds(tiles, planes, per_cu, c);
    if (masked) rounds += (blocks / 2 + cap - 1) / cap + (3 * blocks / 4 + cap - 1) / cap;
    const int64_t t = rounds * (c + kChunkHead);
    if (t <= cost) { cost = t; best = c; }
  }
  return best;
}

// One thread per cell of the mask.
__global__ __launch_bounds__(256) void k_sg_mask_cells(const SgConvParams p) {
  const int64_t cy = sg_cells(p.ny), cx = sg_cells(p.nx);
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= sg_cells(p.nz) * cy * cx) return;
  if (i == 0) *p.work = 0;
  const int64_t x0 = i % cx * kSgCell, y0 = i / cx % cy * kSgCell, z0 = i / (cx * cy) * kSgCell;
  uint32_t any = 0;
#pragma unroll
  for (int r = 0; r < kSgCell * kSgCell; ++r) {
    const int64_t z = clampi(z0 + r / kSgCell, p.nz), y = clampi(y0 + r % kSgCell, p.ny);
    const uint8_t* row = p.mask + (z * p.ny + y) * p.nx;
#pragma unroll
    for (int k = 0; k < kSgCell; ++k) any |= row[clampi(x0 + k, p.nx)];
  }
  p.cells[i] = any != 0;
}

// A mask gates the outputs, so a layer is needed only within reach of a masked
// voxel: on a wall that fills 0.41 of 256 x 320 x 384 the five layers take 5.0 ms
// instead of 6.7.
// Narrows planes [z0, z1) of the tile of ty x tx voxels at (y0, x0) to those within
// p.reach voxels of a marked cell (none: z1 = z0).  Every thread of the block
// calls it; lds: two ints.
__device__ __forceinline__ void masked_planes(const SgConvParams& p, int64_t y0, int64_t x0, int ty, int tx,
                                              int64_t& z0, int64_t& z1, int* lds) {
  if (p.cells == nullptr) return;  // kernel argument: uniform
  const int d = p.reach;
  const int64_t cy = sg_cells(p.ny), cx = sg_cells(p.nx);
  const int ya = static_cast<int>(clampi(y0 - d, p.ny)) / kSgCell, yb = static_cast<int>(clampi(y0 + ty - 1 + d, p.ny)) / kSgCell;
  const int xa = static_cast<int>(clampi(x0 - d, p.nx)) / kSgCell, xb = static_cast<int>(clampi(x0 + tx - 1 + d, p.nx)) / kSgCell;
  const int za = static_cast<int>(clampi(z0 - d, p.nz)) / kSgCell, zb = static_cast<int>(clampi(z1 - 1 + d, p.nz)) / kSgCell;
  if (threadIdx.x == 0) {
    lds[0] = zb + 1;
    lds[1] = za - 1;
  }
  __syncthreads();
  const int wy = yb - ya + 1, wx = xb - xa + 1;
  int lo = zb + 1, hi = za - 1;
  for (int i = threadIdx.x; i < (zb - za + 1) * wy * wx; i += blockDim.x) {
    const int z = za + i / (wy * wx), y = ya + i / wx % wy, x = xa + i % wx;
    if (p.cells[(z * cy + y) * cx + x] != 0) {
      lo = min(lo, z);
      hi = max(hi, z);
    }
  }
  if (lo <= hi) {
    atomicMin(&lds[0], lo);
    atomicMax(&lds[1], hi);
  }
  __syncthreads();
  lo = lds[0];
  hi = lds[1];
  z1 = lo <= hi ? min(z1, static_cast<int64_t>(kSgCell) * hi + kSgCell + d) : z0;
  z0 = lo <= hi ? max(z0, static_cast<int64_t>(kSgCell) * lo - d) : z0;
}

// First layer: the input is the raw volume, one channel.
template <typename Tin>
__global__ __launch_bounds__(NT) void k_sg_conv(const SgConvParams p) {
  __shared__ __attribute__((aligned(16))) __bf16 wl[C * 32];
  __shared__ __bf16 al[3 * PLANE_VOX];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t b = blockIdx.x;
  const int64_t xt = b % p.x_tiles;
  b /= p.x_tiles;
  const int64_t yt = b % p.y_tiles;
  const int64_t zc = b / p.y_tiles;
  const int64_t x0 = xt * TX, y0 = yt * TY;
  const int64_t nz = p.nz, ny = p.ny, nx = p.nx;
  int64_t z0 = p.z_lo + zc * p.zchunk;
  int64_t z1 = (z0 + p.zchunk) < p.z_hi ? (z0 + p.zchunk) : p.z_hi;
  __shared__ int planes[2];
  masked_planes(p, y0, x0, TY, TX, z0, z1, planes);
  if (z0 >= z1) return;  // block-uniform
  if (p.work != nullptr && tid == 0) atomicAdd(p.work, static_cast<int>(z1 - z0));

  // weights: 16-byte chunks
  {
    const bf16x8* src = reinterpret_cast<const bf16x8*>(p.w1);
    bf16x8* dst = reinterpret_cast<bf16x8*>(wl);
    for (int i = tid; i < C * 32 / 8; i += NT) dst[i] = src[i];
  }

  const double in_scale = static_cast<double>(p.scale_offset[0]);
  const double in_offset = static_cast<double>(p.scale_offset[1]);

  // staging of one input plane (index zi, clamped): one value per voxel
  constexpr int PER = (PLANE_VOX + NT - 1) / NT;
  static_assert(PER == 1, "one staged value per thread");
  const int vi = tid < PLANE_VOX ? tid : PLANE_VOX - 1;
  const int64_t off = clampi(y0 - 1 + vi / RX, ny) * nx + clampi(x0 - 1 + vi % RX, nx);
  auto load_plane = [&](int64_t zi) {
    return static_cast<float>(static_cast<const Tin*>(p.vol)[clampi(zi, nz) * ny * nx + off]);
  };
  auto store_plane = [&](int s, float v) {
    if (tid < PLANE_VOX)  // float64 affine map (exact product, one rounding), then float32, then bf16
      al[s * PLANE_VOX + tid] =
          static_cast<__bf16>(static_cast<float>(fma(static_cast<double>(v), in_scale, in_offset)));
  };

  store_plane(0, load_plane(z0 - 1));
  store_plane(1, load_plane(z0));
  store_plane(2, load_plane(z0 + 1));
  __syncthreads();

  const int li = lane & 15, lk = lane >> 4;
  const int64_t yo = y0 + wave;
  float bias[2][4];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) bias[m][r] = p.bias[16 * m + 4 * lk + r];
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), as in k_sg_conv_ws
#pragma unroll 1
  for (int64_t z = z0; z < z1; ++z) {
    // ring slot of input plane z + d is (z - z0 + 1 + d) mod 3
    const int s0 = static_cast<int>((z - z0) % 3);  // plane z - 1
    const bool more = z + 1 < z1;
    float pv = 0.f;
    if (more) pv = load_plane(z + 2);  // in flight during the products

    f32x4 acc[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

    // K = 32 "taps" of the single input channel (27 real, 5 zero)
    bf16x8 bo[2];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = 8 * lk + i;
        if (k < 27) {
          const int dz = k / 9, dy = (k / 3) % 3, dx = k % 3;  // offsets + 1
          const int s = (s0 + dz) % 3;
          bo[n][i] = al[s * PLANE_VOX + (wave + dy) * RX + 16 * n + li + dx];
        } else {
          bo[n][i] = static_cast<__bf16>(0.f);
        }
      }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const bf16x8 a = reinterpret_cast<const bf16x8*>(wl)[(16 * m + li) * 4 + lk];
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bo[n], acc[m][n], 0, 0, 0);
    }

#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int64_t xv = x0 + 16 * n + li;
      if (yo < ny && xv < nx) {
        const int64_t vox = ((z - p.out_z0) * ny + yo) * nx + xv;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int co = 16 * m + 4 * lk;
          bf16x4 o;
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] = static_cast<__bf16>(fmaxf(acc[m][n][r] + bias[m][r], 0.f));
          *reinterpret_cast<bf16x4*>(p.out + vox * C + co) = o;
        }
      }
    }

    __syncthreads();  // every read of the ring slot about to be replaced is done
    if (more) {
      store_plane(s0, pv);  // plane z + 2 replaces plane z - 1
      __syncthreads();
    }
  }
}

// Weight-stationary 32 -> 32 layer: inference layers 2..5 and the training
// passes.  A block of 4 waves (one per SIMD) owns 16 (y) x 32 (x) output voxels
// and marches through a chunk of z planes; wave w computes rows 4w .. 4w + 3, i.e.
// eight 16-voxel N blocks.  Every lane holds its A operands of all 27 taps and
// both 16-channel M blocks in registers for the whole chunk (216 VGPRs: the
// layer's weights are read from memory once per block), so per tap the wave reads
// only its B operands from the LDS ring and issues 16 MFMAs.  The input planes
// live in a ring of 3 LDS planes of 18 rows (faces clamped; 135 KB, one block per
// CU); the next plane's loads are issued before the current plane's products
// and stored into the ring right after them, before the epilogue.  Four rows of
// 32 a wave, against two of 64, let the taps of neighbouring rows share more
// operands (108 LDS reads a plane for 216 operands, against 144) and stage 1.20
// instead of 1.29 voxels per output.
//
// A lane's operand is 16 bytes (8 channels: piece lk of a voxel's four).  A
// 16-byte LDS read is served 16 lanes at a time (lanes 0-3, 12-15 and 20-27 of the
// first 32, then the other 16, and so on) over 64 banks; with voxels of 64 bytes
// laid out plainly, two lanes of such a group meet in every bank.  The pieces of
// a voxel are therefore exchanged in pairs (piece p at place p ^ 2) where bit 2
// of the voxel's place is set, which parts them for any first voxel.  Rows are
// WS_RXP = 40 places, a multiple of 8, so that bit depends only on the lane and
// the tap's x offset and every other offset stays an instruction immediate.
//
// MODE: WS_HIDDEN stores the activation; WS_LAST evaluates the head as three more
// MFMAs per N block (the layer's output and the head weights each split into a
// high and a low bf16 part, about 16 bits of each, all products but low x low);
// WS_BWD is the backward data pass (no bias, the output multiplied by the ReLU
// mask of p.prev, the forward activation at the output voxel).
//
// What bounds it: the matrix cores at the clock their power leaves (60 % of the
// cycles busy at about 2.0 GHz: 1.23 PFLOP/s, a large library product reaches
// 1.1 to 1.4 on this card); one wave per SIMD leaves the epilogue uncovered.
// A hidden layer of 256 x 320 x 384 takes 1420 us (1530 with two rows of 64 a wave,
// plain piece order and 8-byte stores), the last layer 2100 (2217), the training
// layers of 32 patches of 32^3 57 forward and 68 backward (78 and 86 with
// the weights streamed from LDS).
constexpr int WS_RW = 4, WS_NB = 2;  // rows per wave, 16-voxel blocks per row
constexpr int WS_TY = 4 * WS_RW, WS_TX = 16 * WS_NB, WS_RY = WS_TY + 2, WS_RX = WS_TX + 2;
constexpr int WS_RXP = (WS_RX + 7) / 8 * 8;
constexpr int WS_NT = 256;
constexpr int WS_PLANE = WS_RY * WS_RXP;                          // places of one staged plane
constexpr int WS_PIECES = WS_RY * WS_RX * 4;                      // 16-byte pieces of one staged plane
constexpr int WS_PER = (WS_PIECES + WS_NT - 1) / WS_NT;           // per thread
constexpr int WS_HIDDEN = 0, WS_LAST = 1, WS_BWD = 2;

// Zeros every output of the tile at (y0, x0) in planes [za, zb).
__device__ __forceinline__ void zero_outputs(const SgConvParams& p, int64_t y0, int64_t x0, int64_t za, int64_t zb) {
  const int64_t x = x0 + threadIdx.x % WS_TX;
  if (x >= p.nx) return;
  for (int64_t z = za; z < zb; ++z)
    for (int r = threadIdx.x / WS_TX; r < WS_TY && y0 + r < p.ny; r += WS_NT / WS_TX) {
      const int64_t vox = (z * p.ny + y0 + r) * p.nx + x;
      if (p.e3) { p.e3[vox] = 0.f; p.e3[p.n + vox] = 0.f; p.e3[2 * p.n + vox] = 0.f; }
      if (p.fa) p.fa[vox] = 0.f;
      if (p.conf) p.conf[vox] = 0.f;
      if (p.ha) p.ha[vox] = 0.f;
      if (p.ia) p.ia[vox] = 0.f;
    }
}

template <int MODE>
__global__ __launch_bounds__(WS_NT) void k_sg_conv_ws(const SgConvParams p) {
  constexpr bool LAST = MODE == WS_LAST;
  __shared__ __attribute__((aligned(16))) __bf16 al[3 * WS_PLANE * C];
  __shared__ float hw[LAST ? 5 * C : 1];  // head weights (read by lane-dependent channel)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  if constexpr (LAST) {
    if (tid < 5 * C) hw[tid] = p.head_w[tid];
  }
  const int64_t nz = p.nz, ny = p.ny, nx = p.nx;
  int64_t b = blockIdx.x;
  const int64_t xt = b % p.x_tiles;
  b /= p.x_tiles;
  const int64_t yt = b % p.y_tiles;
  const int64_t zc = b / p.y_tiles;
  const int64_t x0 = xt * WS_TX, y0 = yt * WS_TY;
  const int64_t zchunk = p.work != nullptr && *p.work <= p.few ? p.zchunk_few : p.zchunk;
  int64_t z0 = p.z_lo + zc * zchunk;
  if (z0 >= p.z_hi) return;  // the grid is that of the shorter chunks
  int64_t z1 = (z0 + zchunk) < p.z_hi ? (z0 + zchunk) : p.z_hi;
  {
    __shared__ int planes[2];
    const int64_t za = z0, zb = z1;
    masked_planes(p, y0, x0, WS_TY, WS_TX, z0, z1, planes);
    if constexpr (LAST) {  // no voxel of the mask in the other planes
      zero_outputs(p, y0, x0, za, z0);
      zero_outputs(p, y0, x0, z1, zb);
    }
    if (z0 >= z1) return;  // block-uniform
  }

  // the thread's staged pieces: place in the volume's plane (voxels, below 2^31
  // since a plane of activations is 64 bytes a voxel) and in the ring's
  int goff[WS_PER], loff[WS_PER];
#pragma unroll
  for (int j = 0; j < WS_PER; ++j) {
    int c = tid + WS_NT * j;
    if (c >= WS_PIECES) c = WS_PIECES - 1;  // the last piece again
    const int row = (c >> 2) / WS_RX, col = (c >> 2) % WS_RX, part = c & 3;
    goff[j] = static_cast<int>(clampi(y0 - 1 + row, ny) * nx + clampi(x0 - 1 + col, nx));
    loff[j] = (row * WS_RXP + col) * 4 + (part ^ (((col >> 2) & 1) << 1));
  }
  auto load_plane = [&](int64_t zi, bf16x8 (&pf)[WS_PER]) {
    const __bf16* src = p.in + (clampi(zi, nz) - p.in_z0) * ny * nx * C + 8 * (tid & 3);
#pragma unroll
    for (int j = 0; j < WS_PER; ++j)
      pf[j] = *reinterpret_cast<const bf16x8*>(src + static_cast<int64_t>(goff[j]) * C);
  };
  auto store_plane = [&](int s, const bf16x8 (&pf)[WS_PER]) {
    bf16x8* dst = reinterpret_cast<bf16x8*>(al) + s * WS_PLANE * 4;
#pragma unroll
    for (int j = 0; j < WS_PER; ++j)
      if (tid + WS_NT * j < WS_PIECES) dst[loff[j]] = pf[j];
  };

  bf16x8 pf[WS_PER], pf1[WS_PER], pf2[WS_PER];
  load_plane(z0 - 1, pf);
  load_plane(z0, pf1);
  load_plane(z0 + 1, pf2);
  // Output channel of row i of M block m.  A stored layer deals the channels to
  // the two blocks in fours, so that a lane's eight results (rows 4 lk .. 4 lk + 3
  // of both) are the neighbouring channels 8 lk .. 8 lk + 7: one 16-byte store.
  // The last layer keeps them in order, as the head's columns are.
  auto channel = [](int m, int i) { return LAST ? 16 * m + i : 8 * (i >> 2) + 4 * m + (i & 3); };
  // A operands: lane holds W[t][channel(m, li)][8 lk .. 8 lk + 7]
  bf16x8 wa[27][2];
  {
    const bf16x8* w8 = reinterpret_cast<const bf16x8*>(p.w);
#pragma unroll
    for (int t = 0; t < 27; ++t)
#pragma unroll
      for (int m = 0; m < 2; ++m) wa[t][m] = w8[(t * C + channel(m, li)) * 4 + lk];
  }
  float bias[2][4];
  if constexpr (MODE != WS_BWD) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) bias[m][r] = p.bias[channel(m, 4 * lk + r)];
  }
  store_plane(0, pf);
  store_plane(1, pf1);
  store_plane(2, pf2);
  __syncthreads();
  // The weights and biases arrive before the plane loop: vector memory counts
  // loads and stores together, so a load that may still be pending at the loop's
  // head makes every use of it wait, in every plane, for stores just issued.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)

  // LAST: the head h = Wh x5 on the matrix cores, with Wh (rows 0..4 of a
  // 16-row A operand) split into a bf16 high and low part.  A lane's B operand
  // is its own eight channels of x5, so its K index 8 lk + i stands for
  // channel 16 (i / 4) + 4 lk + i % 4, and A's columns follow that order.
  bf16x8 wh_hi, wh_lo;
  float hb[5];  // read here once: after the first store they would be read for every voxel
  if constexpr (LAST) {
#pragma unroll
    for (int q = 0; q < 5; ++q) hb[q] = p.head_b[q];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float wv = li < 5 ? hw[li * C + 16 * (i >> 2) + 4 * lk + (i & 3)] : 0.f;
      const __bf16 hi = static_cast<__bf16>(wv);
      wh_hi[i] = hi;
      wh_lo[i] = static_cast<__bf16>(wv - static_cast<float>(hi));
    }
  }

  const bf16x8* a8 = reinterpret_cast<const bf16x8*>(al);
  int at[3];  // this lane's operand of the wave's first row, by the tap's x offset
#pragma unroll
  for (int dx = 0; dx < 3; ++dx)
    at[dx] = (WS_RW * wave * WS_RXP + li + dx) * 4 + (lk ^ ((((li + dx) >> 2) & 1) << 1));
#pragma unroll 1
  for (int64_t z = z0; z < z1; ++z) {
    const int s0 = static_cast<int>((z - z0) % 3);  // ring slot of plane z - 1
    const bool more = z + 1 < z1;
    if (more) load_plane(z + 2, pf);  // in flight during the products
    // what the epilogue reads, too (clamped: of a voxel outside, nothing is stored)
    bf16x8 xm[MODE == WS_BWD ? 8 : 1];
    uint8_t inside[2] = {1, 1};
    if constexpr (MODE == WS_BWD) {
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        const int64_t yo = clampi(y0 + WS_RW * wave + n / WS_NB, ny), xv = clampi(x0 + 16 * (n % WS_NB) + li, nx);
        xm[n] = *reinterpret_cast<const bf16x8*>(p.prev + (((z - p.out_z0) * ny + yo) * nx + xv) * C + 8 * lk);
      }
    }
    if constexpr (LAST) {
      if (p.mask != nullptr) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int n = 4 * k + lk;
          const int64_t yo = clampi(y0 + WS_RW * wave + n / WS_NB, ny), xv = clampi(x0 + 16 * (n % WS_NB) + li, nx);
          inside[k] = p.mask[(z * ny + yo) * nx + xv];
        }
      }
    }

    // ring planes z - 1, z, z + 1; row and N-block offsets are immediates
    const bf16x8* base[3];
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) base[dz] = a8 + (s0 + dz) % 3 * WS_PLANE * 4;
    // products of NB N blocks from block n0 on, every tap into one chain per result
    auto products = [&]<int NB>(std::integral_constant<int, NB>, int n0, f32x4 (&acc)[2][NB]) {
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 27; ++t) {
        const int dz = t / 9, dy = (t / 3) % 3, dx = t % 3;
        bf16x8 bo[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n)
          bo[n] = (base[dz] + at[dx])[(((n0 + n) / WS_NB + dy) * WS_RXP + 16 * ((n0 + n) % WS_NB)) * 4];
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
          for (int m = 0; m < 2; ++m)
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[t][m], bo[n], acc[m][n], 0, 0, 0);
      }
    };

    if constexpr (!LAST) {
      f32x4 acc[2][8];
      products(std::integral_constant<int, 8>{}, 0, acc);
      // the prefetched plane goes into the ring before the epilogue, so its
      // registers are free there
      __syncthreads();  // every read of the ring slot about to be replaced is done
      if (more) store_plane(s0, pf);  // plane z + 2 replaces plane z - 1
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        const int64_t yo = y0 + WS_RW * wave + n / WS_NB, xv = x0 + 16 * (n % WS_NB) + li;
        if (yo < ny && xv < nx) {
          const int64_t vox = ((z - p.out_z0) * ny + yo) * nx + xv;
          bf16x8 o;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float v = acc[i >> 2][n][i & 3];
            if constexpr (MODE == WS_BWD)
              o[i] = static_cast<__bf16>(static_cast<float>(xm[n][i]) > 0.f ? v : 0.f);
            else
              o[i] = static_cast<__bf16>(fmaxf(v + bias[i >> 2][i & 3], 0.f));
          }
          *reinterpret_cast<bf16x8*>(p.out + vox * C + 8 * lk) = o;
        }
      }
    } else {
      // in two halves of four N blocks, which keeps the outputs' arithmetic out of
      // scratch memory (with all eight blocks' sums live it spills, and every
      // reload waits for the stores before it)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        f32x4 acc[2][4];
        products(std::integral_constant<int, 4>{}, 4 * k, acc);
        if (k == 1) {
          __syncthreads();  // every read of the ring slot about to be replaced is done
          if (more) store_plane(s0, pf);  // plane z + 2 replaces plane z - 1
        }
        // head: x5 = relu(acc + b), split like Wh into a high and a low bf16
        // part, is the B operand as the lane holds it (the product of the two
        // low parts, below 2^-16 of a term, is left out); D row q, column li is
        // h[q] of voxel li (rows 0..3 in lanes 0..15, row 4 in lanes 16..31).
        // Lanes of group lk then finish the voxels of the half's N block lk.
        float o[5];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          bf16x8 xh, xl;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float v = fmaxf(acc[i >> 2][n][i & 3] + bias[i >> 2][i & 3], 0.f);
            xh[i] = static_cast<__bf16>(v);
            xl[i] = static_cast<__bf16>(v - static_cast<float>(xh[i]));
          }
          f32x4 d = f32x4{0.f, 0.f, 0.f, 0.f};
          d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh_hi, xh, d, 0, 0, 0);
          d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh_hi, xl, d, 0, 0, 0);
          d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh_lo, xh, d, 0, 0, 0);
#pragma unroll
          for (int q = 0; q < 5; ++q) {
            const float qv = q < 4 ? __shfl(d[q], li) : __shfl(d[0], 16 + li);
            o[q] = n == 0 || n == lk ? qv : o[q];
          }
        }
        const int n = 4 * k + lk;
        const int64_t yo = y0 + WS_RW * wave + n / WS_NB, xv = x0 + 16 * (n % WS_NB) + li;
        if (yo < ny && xv < nx) {
#pragma unroll
          for (int q = 0; q < 5; ++q) o[q] = hb[q] + o[q];
          head_outputs(p, o, inside[k] != 0, z, yo, xv);
        }
      }
    }

    __syncthreads();  // the replaced slot is written before the next plane's products
  }
}

template <int MODE>
hipError_t launch_conv_ws(const SgConvParams& q, hipStream_t stream) {
  SgConvParams p = q;
  p.x_tiles = (p.nx + WS_TX - 1) / WS_TX;
  p.y_tiles = (p.ny + WS_TY - 1) / WS_TY;
  const int64_t planes = p.z_hi - p.z_lo, tiles = p.x_tiles * p.y_tiles;
  p.zchunk = sg_zchunk(tiles, planes, 1, 64, false);
  int64_t chunks = (planes + p.zchunk - 1) / p.zchunk;
  if (p.work != nullptr) {
    // Shorter chunks fill the chip where a mask leaves few tiles with work, and cost
    // another round where it leaves most of them.  Which holds is known on the device
    // only, so the kernel picks (128^3: a ring 525 us with the short chunks, 490 so, a
    // full mask 549 and 504; a ring in 316 x 48 x 143 347, 520 with the long ones).
    p.zchunk_few = sg_zchunk(tiles, planes, 1, 64, true);
    const auto cost = [&](int64_t t, int64_t c) { return sg_rounds(t, planes, 1, c) * (c + kChunkHead); };
    int64_t few = tiles;  // the most tiles with work for which they are the better
    while (few > 0 && cost(few, p.zchunk_few) >= cost(few, p.zchunk)) --few;
    const int64_t per_tile = p.work_planes * (WS_TY / TY);  // of layer 1's tiles, half as high
    p.few = few > 0 ? static_cast<int>(std::min<int64_t>(few * per_tile, INT32_MAX)) : -1;
    if (few > 0) chunks = std::max(chunks, (planes + p.zchunk_few - 1) / p.zchunk_few);
  }
  const int64_t blocks = tiles * chunks;
  hipLaunchKernelGGL(k_sg_conv_ws<MODE>, dim3(static_cast<unsigned>(blocks)), dim3(WS_NT), 0, stream, p);
  return hipGetLastError();
}

// Voxels inside the mask whose confidence is below the threshold take the
// structure-tensor path's outputs.  A thread takes four voxels 256 apart and issues
// their reads together (first what decides, then what is copied).
constexpr int kMergePer = 4;
__global__ __launch_bounds__(256) void k_sg_merge(const SgMergeParams p) {
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * (256 * kMergePer) + threadIdx.x;
  bool take[kMergePer];
  float conf[kMergePer];
  uint8_t inside[kMergePer];
#pragma unroll
  for (int v = 0; v < kMergePer; ++v) {
    const int64_t t = t0 + 256 * v < p.count ? t0 + 256 * v : p.count - 1;
    conf[v] = p.conf[p.begin + t];
    inside[v] = p.mask == nullptr ? 1 : p.mask[p.begin + t];
  }
  float o[kMergePer][6];
#pragma unroll
  for (int v = 0; v < kMergePer; ++v) {
    take[v] = t0 + 256 * v < p.count && inside[v] != 0 && conf[v] < p.threshold;
    const int64_t j = p.begin + t0 + 256 * v - p.src_shift;
    if (take[v]) {
      if (p.e3) { o[v][0] = p.pe3[j]; o[v][1] = p.pe3[p.src_n + j]; o[v][2] = p.pe3[2 * p.src_n + j]; }
      if (p.fa) o[v][3] = p.pfa[j];
      if (p.ha) o[v][4] = p.pha[j];
      if (p.ia) o[v][5] = p.pia[j];
    }
  }
#pragma unroll
  for (int v = 0; v < kMergePer; ++v) {
    const int64_t i = p.begin + t0 + 256 * v;
    if (take[v]) {
      if (p.e3) { p.e3[i] = o[v][0]; p.e3[p.n + i] = o[v][1]; p.e3[2 * p.n + i] = o[v][2]; }
      if (p.fa) p.fa[i] = o[v][3];
      if (p.ha) p.ha[i] = o[v][4];
      if (p.ia) p.ia[i] = o[v][5];
    }
  }
}

hipError_t launch_first(const SgConvParams& q, int dtype, hipStream_t stream) {
  SgConvParams p = q;
  p.x_tiles = (p.nx + TX - 1) / TX;
  p.y_tiles = (p.ny + TY - 1) / TY;
  const int64_t planes = p.z_hi - p.z_lo;
  if (p.cells != nullptr && p.build_cells) {
    const int64_t cells = sg_cells(p.nz) * sg_cells(p.ny) * sg_cells(p.nx);
    hipLaunchKernelGGL(k_sg_mask_cells, dim3(static_cast<unsigned>((cells + 255) / 256)), dim3(256), 0, stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  p.zchunk = sg_zchunk(p.x_tiles * p.y_tiles, planes, 4, 16, p.cells != nullptr);  // short chunks: the launch ends evenly
  const int64_t blocks = p.x_tiles * p.y_tiles * ((planes + p.zchunk - 1) / p.zchunk);
  if (dtype == ST_DTYPE_U16)
    hipLaunchKernelGGL(k_sg_conv<uint16_t>, dim3(static_cast<unsigned>(blocks)), dim3(NT), 0, stream, p);
  else
    hipLaunchKernelGGL(k_sg_conv<float>, dim3(static_cast<unsigned>(blocks)), dim3(NT), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_sg_pack(const float* blob, __bf16* w1, __bf16* w25, hipStream_t stream) {
  const int64_t n = 4 * 27 * C * C;
  hipLaunchKernelGGL(k_sg_pack, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, blob, w1, w25);
  return hipGetLastError();
}

hipError_t launch_sg_conv(int layer, int dtype, const SgConvParams& p, hipStream_t stream) {
  if (layer == 1) return launch_first(p, dtype, stream);
  if (layer == kSgLayers) return launch_conv_ws<WS_LAST>(p, stream);
  return launch_conv_ws<WS_HIDDEN>(p, stream);
}

hipError_t launch_sg_conv_hidden(bool first, int dtype, const SgConvParams& p, hipStream_t stream) {
  return first ? launch_first(p, dtype, stream) : launch_conv_ws<WS_HIDDEN>(p, stream);
}

hipError_t launch_sg_conv_bwd(const SgConvParams& p, hipStream_t stream) {
  return launch_conv_ws<WS_BWD>(p, stream);
}

hipError_t launch_sg_merge(const SgMergeParams& p, hipStream_t stream) {
  const int64_t per = 256 * kMergePer;
  if (p.count < 1 || (p.count + 255) / 256 > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_sg_merge, dim3(static_cast<unsigned>((p.count + per - 1) / per)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace st
