// Training kernels of the learned orientation surrogate: the loss and the head's
// backward pass, the weight gradients of the five convolutions (on the bf16
// matrix cores), deterministic reductions of per-block partial sums, and Adam
// on the float32 weights.  The forward
// pass and the backward data pass reuse the inference convolution kernel.
//
// Training runs on a stack of P^3 patches, P <= 32, laid out as one volume of
// npatch * P planes of P x P voxels; a row of the stack (fixed z, y) holds the
// P voxels of one MFMA K step.  Activations x_l and gradients g_l (at the
// pre-activation of layer l) are channel-last bf16, [N][32].
#include "st_device.h"
#include "st_surrogate.h"

namespace st {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int C = kSgChannels;
constexpr int WX = kSgTrainMaxX;   // voxels of a staged row
constexpr float kConfDeg = 2.0f;   // confidence target: within this angle of the label

__device__ __forceinline__ int64_t clampi(int64_t v, int64_t n) { return v < 0 ? 0 : (v >= n ? n - 1 : v); }

// Backward weights of layers 2..5: [layer][tap'][a][b] = W[b][a][26 - tap'], so
// that the forward kernel, which reads its weights as [tap][out][in], computes
// dx[a](q) = sum_{b, tap} W[b][a][tap] g[b](q - off(tap)).
__global__ void k_sg_pack_bwd(const float* blob, __bf16* w25t) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t per = 27 * C * C;
  if (i >= 4 * per) return;
  const int layer = static_cast<int>(i / per);
  const int64_t r = i % per;
  const int tp = static_cast<int>(r / (C * C)), a = static_cast<int>((r / C) % C), b = static_cast<int>(r % C);
  w25t[i] = static_cast<__bf16>(blob[kSgOffW2 + layer * kSgLayerStride + (b * C + a) * 27 + (26 - tp)]);
}

// The head and the loss on every weighted voxel: h = bh + Wh x5, direction term
// 1 - (u.t)^2 with u = h[0:3] / |h[0:3]|, FA term (sigmoid(h3) - f)^2, confidence
// term softplus(h4) - c h4 with c = [angle(u, t) < 2 deg].  dL/dh (unnormalised)
// goes back through the head into g5; the head's weight gradient, its bias
// gradient and the six loss sums are one small product over the voxels,
// [11 quantities] x [32 channels and a one], on the float32 matrix cores: a wave
// multiplies the 64 voxels its own lanes evaluated (v_mfma_f32_16x16x4_f32, four
// voxels a step), so no block barrier separates the two, and keeps the sums in
// registers over all its voxels.  Bound by reading x5 and writing g5 (128 bytes
// a voxel) and the per-voxel chain; one thread per sum walking the block's voxels
// in LDS, as before, took 128 us for 2^20 voxels, against 66.
__global__ __launch_bounds__(256) void k_sg_head_train(const SgHeadParams p) {
  constexpr int DS = kSgHeadRow;
  __shared__ __bf16 xs[256][C + 2];
  __shared__ float ds[256 * DS];
  // the head's weights by channel, read by every lane at once: as scalars the
  // 160 do not fit the scalar registers and are loaded anew for every voxel
  __shared__ __attribute__((aligned(16))) float hw[C][8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  f32x4 acc[3];  // channels 0..15, 16..31, the column of ones
#pragma unroll
  for (int n = 0; n < 3; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (tid < 5 * C) hw[tid % C][tid / C] = p.head_w[tid];
  for (int i = tid; i < 256 * DS; i += 256) ds[i] = 0.f;
  __syncthreads();
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * 256; base < p.n;
       base += static_cast<int64_t>(gridDim.x) * 256) {  // block-uniform trip count
    const int64_t v = base + tid;
    float d[11];
    bf16x8 x8[4];
#pragma unroll
    for (int k = 0; k < 11; ++k) d[k] = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) x8[q] = bf16x8{};
    const bool counts = v < p.n && p.weight[v] != 0;
    if (v < p.n) {
      bf16x8 g8[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) g8[q] = bf16x8{};
      if (counts) {
        const bf16x8* src = reinterpret_cast<const bf16x8*>(p.x5 + v * C);
#pragma unroll
        for (int q = 0; q < 4; ++q) x8[q] = src[q];
        float h[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) h[q] = p.head_b[q];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const float4 w4 = *reinterpret_cast<const float4*>(hw[c]);
          const float xc = static_cast<float>(x8[c / 8][c % 8]);
          h[0] = fmaf(w4.x, xc, h[0]);
          h[1] = fmaf(w4.y, xc, h[1]);
          h[2] = fmaf(w4.z, xc, h[2]);
          h[3] = fmaf(w4.w, xc, h[3]);
          h[4] = fmaf(hw[c][4], xc, h[4]);
        }
        const float tz = p.target[v], ty = p.target[p.n + v], tx = p.target[2 * p.n + v];
        const float nrm = sqrtf(h[0] * h[0] + h[1] * h[1] + h[2] * h[2]);
        const float inv = nrm > 0.f ? 1.f / nrm : 1.f;
        const float uz = h[0] * inv, uy = h[1] * inv, ux = h[2] * inv;
        const float dot = uz * tz + uy * ty + ux * tx;
        const float l_dir = 1.f - dot * dot;
        d[0] = -2.f * dot * (tz - dot * uz) * inv;
        d[1] = -2.f * dot * (ty - dot * uy) * inv;
        d[2] = -2.f * dot * (tx - dot * ux) * inv;
        const float s3 = 1.f / (1.f + expf(-h[3]));
        const float e = s3 - p.target_fa[v];
        d[3] = 2.f * e * s3 * (1.f - s3);
        const float cz = uy * tx - ux * ty, cy = ux * tz - uz * tx, cx = uz * ty - uy * tz;
        const float ang = atan2f(sqrtf(cz * cz + cy * cy + cx * cx), fabsf(dot)) * 57.29577951308232f;
        const float c = ang < kConfDeg ? 1.f : 0.f;
        const float s4 = 1.f / (1.f + expf(-h[4]));
        d[4] = p.w_conf * (s4 - c);
        d[5] = l_dir;
        d[6] = e * e;
        d[7] = fmaxf(h[4], 0.f) + log1pf(expf(-fabsf(h[4]))) - c * h[4];
        d[8] = 1.f;
        d[9] = c;
        d[10] = ang;
#pragma unroll
        for (int cc = 0; cc < C; ++cc) {
          const float4 w4 = *reinterpret_cast<const float4*>(hw[cc]);
          float gc = fmaf(w4.x, d[0], 0.f);
          gc = fmaf(w4.y, d[1], gc);
          gc = fmaf(w4.z, d[2], gc);
          gc = fmaf(w4.w, d[3], gc);
          gc = fmaf(hw[cc][4], d[4], gc);
          g8[cc / 8][cc % 8] = static_cast<__bf16>(static_cast<float>(x8[cc / 8][cc % 8]) > 0.f ? gc : 0.f);
        }
      }
      bf16x8* dst = reinterpret_cast<bf16x8*>(p.g5 + v * C);
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[q] = g8[q];
    }
    if (!__any(counts)) continue;  // nothing to add (wave-uniform; no block barrier in the loop)
#pragma unroll
    for (int c = 0; c < C; ++c) xs[tid][c] = x8[c / 8][c % 8];
#pragma unroll
    for (int k = 0; k < 11; ++k) ds[sg_head_place(tid, k)] = d[k];
    // the wave reads only its own lanes' rows
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 4
    for (int i = 0; i < 16; ++i) {
      const int row = 64 * wave + 4 * i + lk;
      const float a = ds[sg_head_place(row, li)];  // li > 10: a product row that is not used
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, static_cast<float>(xs[row][li]), acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, static_cast<float>(xs[row][16 + li]), acc[1], 0, 0, 0);
      acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, 1.f, acc[2], 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // the four waves' sums, added in wave order
  __syncthreads();
  float* part = ds;  // [4][3][16][16]
  static_assert(4 * 3 * 256 <= 256 * DS, "the waves' sums fit");
#pragma unroll
  for (int n = 0; n < 3; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[((wave * 3 + n) * 16 + 4 * lk + r) * 16 + li] = acc[n][r];
  __syncthreads();
  if (tid < kSgHeadSums) {
    const int q = tid < 5 * C ? tid / C : tid - 5 * C;
    const int c = tid < 5 * C ? tid % C : 2 * 16;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += part[((w * 3 + c / 16) * 16 + q) * 16 + c % 16];
    p.partial[static_cast<int64_t>(blockIdx.x) * kSgHeadSums + tid] = s;
  }
}

// One operand of v_mfma_f32_16x16x32_bf16 taken across channel-last LDS rows: lane
// l gets channel l % 16 (of the 16 from `base` on) of rows 8 (l / 16) + 0..7, as
// two transposing reads of four rows each.  A transposing read hands lane 4 r + j
// of each 16 lanes 8 bytes of row r and returns to lane i the four rows' element
// i, so `base` is the lane's own address: row 8 (l / 16) + (l % 16) / 4, element
// 4 (l % 4).
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 read_across(const __bf16* base) {
  typedef __attribute__((address_space(3))) s16x4 lds4;
  union { s16x4 h[2]; bf16x8 v; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(base));
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(base + 4 * C));
  return u.v;
}

// The weight-gradient blocks: a block owns WG_TY rows (y) of every plane of its z
// chunk.  The gradient rows and the input rows around them are staged channel-last,
// as they lie in memory (x one voxel beyond the row on each side, indices clamped;
// voxels that no tap of the row needs are zero, as are gradient voxels past
// nx or ny), and the planes of the input form a ring of three.
constexpr int WG_TY = kSgWgradRows, WG_RY = WG_TY + 2, WG_RX = WX + 2;
constexpr int WG_NT = 512;

// Weight gradient of a 32 -> 32 layer: dW[co][ci][tap] = sum_p g(p)[co] x(p + off(tap))[ci]
// and db[co] = sum_p g(p)[co] over the block's voxels: a matrix product whose K
// runs over voxels, so both operands are read across the channel-last rows by
// transposing LDS reads, and a tap's shift along x is only another row address.
// Wave w accumulates taps w, w + 8, w + 16 (and w + 24 for w < 3; the bias, a
// product with ones, for w = 7), four 16 x 16 tiles each.  The next plane's
// loads are in flight during the products.  LDS reads bound it (18 of 512 bytes
// for 14 MFMAs a row and wave); staging each element on its own into three shifted
// channel-major copies, as before, took 1240 us for 2^20 voxels, against 61.
__global__ __launch_bounds__(WG_NT) void k_sg_wgrad(const SgWgradParams p) {
  constexpr int XP = WG_RY * WG_RX * C;  // one staged input plane
  __shared__ __attribute__((aligned(16))) __bf16 xs[3 * XP];
  __shared__ __attribute__((aligned(16))) __bf16 gs[WG_TY * WX * C];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int64_t nz = p.nz;
  const int ny = static_cast<int>(p.ny), nx = static_cast<int>(p.nx);
  const int y_tiles = (ny + WG_TY - 1) / WG_TY, zchunk = static_cast<int>(p.rows_per_block) / WG_TY;
  const int y0 = static_cast<int>(blockIdx.x) % y_tiles * WG_TY;
  const int64_t z0 = static_cast<int64_t>(static_cast<int>(blockIdx.x) / y_tiles) * zchunk;
  const int len = static_cast<int>(nz - z0 < zchunk ? nz - z0 : zchunk);  // planes of the block
  const int ntap = wave < 3 ? 4 : 3;
  f32x4 acc[4][2][2], accb[2];
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    accb[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[i][m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // staging in 16-byte pieces, four a voxel
  constexpr int XN = (WG_RY * WG_RX * 4 + WG_NT - 1) / WG_NT, GN = WG_TY * WX * 4 / WG_NT;
  static_assert(GN * WG_NT == WG_TY * WX * 4, "gradient pieces divide evenly");
  int xoff[XN], goff[GN];
#pragma unroll
  for (int j = 0; j < XN; ++j) {
    int c = tid + WG_NT * j;
    if (c >= WG_RY * WG_RX * 4) c = WG_RY * WG_RX * 4 - 1;
    const int row = (c >> 2) / WG_RX, col = (c >> 2) % WG_RX;
    const int yy = static_cast<int>(clampi(y0 - 1 + row, ny)), xx = static_cast<int>(clampi(col - 1, nx));
    xoff[j] = y0 - 1 + row <= ny && col - 1 <= nx ? (yy * nx + xx) * C + 8 * (c & 3) : -1;
  }
#pragma unroll
  for (int j = 0; j < GN; ++j) {
    const int c = tid + WG_NT * j;
    const int row = (c >> 2) / WX, col = (c >> 2) % WX;
    goff[j] = y0 + row < ny && col < nx ? ((y0 + row) * nx + col) * C + 8 * (c & 3) : -1;
  }
  const int64_t plane = static_cast<int64_t>(ny) * nx * C;
  bf16x8 px[XN], pg[GN];
  auto load_x = [&](int64_t z) {
    const __bf16* src = p.x + clampi(z, nz) * plane;
#pragma unroll
    for (int j = 0; j < XN; ++j) {
      px[j] = bf16x8{};
      if (xoff[j] >= 0) px[j] = *reinterpret_cast<const bf16x8*>(src + xoff[j]);
    }
  };
  auto store_x = [&](int slot) {
#pragma unroll
    for (int j = 0; j < XN; ++j) {
      const int c = tid + WG_NT * j;
      if (c < WG_RY * WG_RX * 4) reinterpret_cast<bf16x8*>(xs + slot * XP)[c] = px[j];
    }
  };
  auto load_g = [&](int64_t z) {
    const __bf16* src = p.g + z * plane;
#pragma unroll
    for (int j = 0; j < GN; ++j) {
      pg[j] = bf16x8{};
      if (goff[j] >= 0) pg[j] = *reinterpret_cast<const bf16x8*>(src + goff[j]);
    }
  };
  load_x(z0 - 1);
  store_x(0);
  load_x(z0);
  store_x(1);
  load_x(z0 + 1);
  load_g(z0);
  const int lane_at = (8 * lk + (li >> 2)) * C + 4 * (li & 3);  // read_across: the lane's own address
  bf16x8 ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = static_cast<__bf16>(1.f);
#pragma unroll 1
  for (int j = 0; j < len; ++j) {  // plane z0 + j; block-uniform trip count
    const int s0 = j % 3;  // ring slot of plane z - 1
    store_x((s0 + 2) % 3);
#pragma unroll
    for (int k = 0; k < GN; ++k) reinterpret_cast<bf16x8*>(gs)[tid + WG_NT * k] = pg[k];
    __syncthreads();
    if (j + 1 < len) {
      load_x(z0 + j + 2);
      load_g(z0 + j + 1);
    }
    int xat[4];  // the taps' first rows in the ring
#pragma unroll
    for (int ti = 0; ti < 4; ++ti) {
      const int t = wave + 8 * ti;
      xat[ti] = ((s0 + t / 9) % 3) * XP + ((t / 3) % 3 * WG_RX + t % 3) * C + lane_at;
    }
    const int rows = ny - y0 < WG_TY ? ny - y0 : WG_TY;
    for (int r = 0; r < rows; ++r) {
      bf16x8 A[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) A[m] = read_across(gs + r * WX * C + lane_at + 16 * m);
#pragma unroll
      for (int ti = 0; ti < 4; ++ti) {
        if (ti < ntap) {  // wave-uniform
          bf16x8 B[2];
#pragma unroll
          for (int n = 0; n < 2; ++n) B[n] = read_across(xs + xat[ti] + r * WG_RX * C + 16 * n);
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n)
              acc[ti][m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[m], B[n], acc[ti][m][n], 0, 0, 0);
        }
      }
      if (wave == 7) {
#pragma unroll
        for (int m = 0; m < 2; ++m) accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[m], ones, accb[m], 0, 0, 0);
      }
    }
    __syncthreads();  // the next plane replaces plane z - 1 and the gradient rows
  }
  float* out = p.partial + static_cast<int64_t>(blockIdx.x) * (27 * C * C + C);
#pragma unroll
  for (int ti = 0; ti < 4; ++ti) {
    if (ti < ntap) {
      const int t = wave + 8 * ti;
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int co = 16 * m + 4 * lk + q, ci = 16 * n + li;
            out[(t * C + co) * C + ci] = acc[ti][m][n][q];
          }
    }
  }
  if (wave == 7 && li == 0) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int q = 0; q < 4; ++q) out[27 * C * C + 16 * m + 4 * lk + q] = accb[m][q];
  }
}

// Weight gradient of layer 1 (one input channel): dW1[co][tap] = sum_p g1(p)[co]
// x0(p + off(tap)) and db1[co] = sum_p g1(p)[co], with x0 = bf16(v * scale + offset)
// formed exactly as the first convolution forms it.  N = the 27 taps and a column
// of ones (the bias), K = a row's voxels; wave w takes row w of the block's
// rows, and the waves' sums are added in wave order at the end.  The gradient is
// read across as above; a tap's operand is eight neighbouring bf16 of one
// staged row.  Reading g bounds it (64 bytes a voxel): 24 us for 2^20 voxels,
// against 475 with one multiply-add per weight and voxel on the vector ALUs.
template <typename Tin>
__global__ __launch_bounds__(WG_NT) void k_sg_wgrad1(const SgWgradParams p) {
  __shared__ __attribute__((aligned(16))) __bf16 gs[WG_TY * WX * C];
  __shared__ __bf16 x0s[3 * WG_RY * WG_RX];
  __shared__ float part[8][4][16 * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int64_t nz = p.nz;
  const int ny = static_cast<int>(p.ny), nx = static_cast<int>(p.nx);
  const int y_tiles = (ny + WG_TY - 1) / WG_TY, zchunk = static_cast<int>(p.rows_per_block) / WG_TY;
  const int y0 = static_cast<int>(blockIdx.x) % y_tiles * WG_TY;
  const int64_t z0 = static_cast<int64_t>(static_cast<int>(blockIdx.x) / y_tiles) * zchunk;
  const int len = static_cast<int>(nz - z0 < zchunk ? nz - z0 : zchunk);  // planes of the block
  const double scale = static_cast<double>(p.scale_offset[0]), offset = static_cast<double>(p.scale_offset[1]);
  const Tin* vol = static_cast<const Tin*>(p.vol);
  constexpr int GN = WG_TY * WX * 4 / WG_NT, XE = WG_RY * WG_RX;
  static_assert(XE <= WG_NT, "one staged input value per thread");
  int goff[GN];
#pragma unroll
  for (int j = 0; j < GN; ++j) {
    const int c = tid + WG_NT * j;
    const int row = (c >> 2) / WX, col = (c >> 2) % WX;
    goff[j] = y0 + row < ny && col < nx ? ((y0 + row) * nx + col) * C + 8 * (c & 3) : -1;
  }
  const int64_t plane = static_cast<int64_t>(ny) * nx;
  const int xe = tid < XE ? tid : XE - 1;
  const int64_t xoff = clampi(y0 - 1 + xe / WG_RX, ny) * nx + clampi(xe % WG_RX - 1, nx);
  bf16x8 pg[GN];
  float pv;
  auto load_g = [&](int64_t z) {
#pragma unroll
    for (int j = 0; j < GN; ++j) {
      pg[j] = bf16x8{};
      if (goff[j] >= 0) pg[j] = *reinterpret_cast<const bf16x8*>(p.g + z * plane * C + goff[j]);
    }
  };
  auto load_x = [&](int64_t z) { pv = static_cast<float>(vol[clampi(z, nz) * plane + xoff]); };
  auto store_x = [&](int slot) {
    if (tid < XE)
      x0s[slot * XE + tid] =
          static_cast<__bf16>(static_cast<float>(fma(static_cast<double>(pv), scale, offset)));
  };
  f32x4 acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  load_x(z0 - 1);
  store_x(0);
  load_x(z0);
  store_x(1);
  load_x(z0 + 1);
  load_g(z0);
  const int lane_at = (8 * lk + (li >> 2)) * C + 4 * (li & 3);
#pragma unroll 1
  for (int j = 0; j < len; ++j) {  // plane z0 + j; block-uniform trip count
    const int s0 = j % 3;
    store_x((s0 + 2) % 3);
#pragma unroll
    for (int k = 0; k < GN; ++k) reinterpret_cast<bf16x8*>(gs)[tid + WG_NT * k] = pg[k];
    __syncthreads();
    if (j + 1 < len) {
      load_x(z0 + j + 2);
      load_g(z0 + j + 1);
    }
    bf16x8 A[2], B[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) A[m] = read_across(gs + wave * WX * C + lane_at + 16 * m);
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int t = 16 * n + li;  // 27: the ones; above: zero
      const int tt = t < 27 ? t : 0;
      const __bf16* src = x0s + ((s0 + tt / 9) % 3) * XE + (wave + (tt / 3) % 3) * WG_RX + tt % 3 + 8 * lk;
#pragma unroll
      for (int i = 0; i < 8; ++i) B[n][i] = t < 27 ? src[i] : static_cast<__bf16>(t == 27 ? 1.f : 0.f);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[m], B[n], acc[m][n], 0, 0, 0);
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[wave][2 * m + n][(4 * lk + q) * 16 + li] = acc[m][n][q];
  __syncthreads();
  constexpr int NJ = C * 27 + C;  // 864 weights [co][tap], 32 biases
  for (int j = tid; j < NJ; j += WG_NT) {
    const int co = j < C * 27 ? j / 27 : j - C * 27, t = j < C * 27 ? j % 27 : 27;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += part[w][2 * (co / 16) + t / 16][(co % 16) * 16 + t % 16];
    p.partial[static_cast<int64_t>(blockIdx.x) * NJ + j] = s;
  }
}

// Sums of the blocks' partials: 64 columns a block, its RED_SEG waves taking every
// RED_SEG-th partial and adding their sums in wave order (a fixed order).  One
// thread per column over all partials, as before, left the loads in one serial
// chain: 61 us for the 256 partials of a layer against 5.8, and 232 us for the
// head's 1024 against 5.2.
constexpr int RED_SEG = 16;
__global__ __launch_bounds__(64 * RED_SEG) void k_sg_reduce(const float* partial, int blocks, int len, int mode,
                                                            float* out) {
  __shared__ float seg[RED_SEG][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = static_cast<int>(blockIdx.x) * 64 + lane;
  float s = 0.f;
  if (j < len) {
#pragma unroll 8
    for (int b = w; b < blocks; b += RED_SEG) s += partial[static_cast<int64_t>(b) * len + j];
  }
  seg[w][lane] = s;
  __syncthreads();
  if (w != 0 || j >= len) return;
#pragma unroll
  for (int q = 1; q < RED_SEG; ++q) s += seg[q][lane];
  int dst = j;
  if (mode == 1) {
    constexpr int NW = 27 * C * C;
    if (j < NW) {
      const int t = j / (C * C), co = (j / C) % C, ci = j % C;
      dst = (co * C + ci) * 27 + t;
    }
  }
  out[dst] = s;
}

// The gradient divided by the weight sum, and the loss means.  raw: the six loss
// sums (dir, fa, conf, weights, within, angle).
__global__ void k_sg_finish(float* grad, int64_t n, const float* raw, float w_conf, float* stats) {
  const float wsum = raw[3];
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    grad[i] = i < 2 ? 0.f : grad[i] * inv;
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const float dir = raw[0] * inv, fa = raw[1] * inv, conf = raw[2] * inv;
  stats[0] = dir;
  stats[1] = fa;
  stats[2] = conf;
  stats[3] = dir + fa + w_conf * conf;
  stats[4] = wsum;
  stats[5] = raw[4];
  stats[6] = raw[5] * inv;
  stats[7] = wsum;
}

__global__ void k_sg_adam(float* w, const float* g, float* m, float* v, int64_t n, int64_t frozen, float lr,
                          float b1, float b2, float eps, float c1, float c2) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < frozen || i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

}  // namespace

hipError_t launch_sg_pack_bwd(const float* blob, __bf16* w25t, hipStream_t stream) {
  const int64_t n = 4 * 27 * C * C;
  hipLaunchKernelGGL(k_sg_pack_bwd, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, blob, w25t);
  return hipGetLastError();
}

hipError_t launch_sg_head_train(const SgHeadParams& p, int blocks, hipStream_t stream) {
  hipLaunchKernelGGL(k_sg_head_train, dim3(blocks), dim3(256), 0, stream, p);
  return hipGetLastError();
}

// The kernels index LDS and the stack by these sizes.
static bool wgrad_ok(const SgWgradParams& p, int blocks) {
  if (p.nx < 1 || p.nx > WX || p.ny < 1 || p.ny > WX || p.nz < 1 || p.rows_per_block < WG_TY ||
      p.rows_per_block % WG_TY != 0)
    return false;
  const int64_t zc = p.rows_per_block / WG_TY;
  return blocks == (p.ny + WG_TY - 1) / WG_TY * ((p.nz + zc - 1) / zc);
}

hipError_t launch_sg_wgrad(const SgWgradParams& p, int blocks, hipStream_t stream) {
  if (!wgrad_ok(p, blocks)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_sg_wgrad, dim3(blocks), dim3(WG_NT), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_sg_wgrad1(int dtype, const SgWgradParams& p, int blocks, hipStream_t stream) {
  if (!wgrad_ok(p, blocks)) return hipErrorInvalidValue;
  if (dtype == ST_DTYPE_U16)
    hipLaunchKernelGGL(k_sg_wgrad1<uint16_t>, dim3(blocks), dim3(WG_NT), 0, stream, p);
  else
    hipLaunchKernelGGL(k_sg_wgrad1<float>, dim3(blocks), dim3(WG_NT), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_sg_reduce(const float* partial, int blocks, int len, int mode, float* out, hipStream_t stream) {
  hipLaunchKernelGGL(k_sg_reduce, dim3(static_cast<unsigned>((len + 63) / 64)), dim3(64 * RED_SEG), 0, stream, partial,
                     blocks, len, mode, out);
  return hipGetLastError();
}

hipError_t launch_sg_finish(float* grad, int64_t n, const float* raw, float w_conf, float* stats, hipStream_t stream) {
  hipLaunchKernelGGL(k_sg_finish, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, grad, n, raw,
                     w_conf, stats);
  return hipGetLastError();
}

hipError_t launch_sg_adam(float* params, const float* grad, float* m, float* v, int64_t n, int64_t frozen,
                          int64_t step, float lr, float beta1, float beta2, float eps, hipStream_t stream) {
  const float c1 = 1.f - powf(beta1, static_cast<float>(step)), c2 = 1.f - powf(beta2, static_cast<float>(step));
  hipLaunchKernelGGL(k_sg_adam, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, params, grad, m,
                     v, n, frozen, lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace st
