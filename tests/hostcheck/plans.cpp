// What the library's host code plans for masked volumes, split passes and the
// re-angling call, checked without a GPU (see hostcheck.h).  The launch functions
// of stub_kernels.cpp are wrapped at link time (--wrap): the checks here come
// first, then that file's own.  One group of checks per run, named by the first
// argument; prints "plans: OK" and exits 0 when all hold.
#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "hostcheck.h"
#include "st.h"
#include "st_host.h"
#include "st_internal.h"
#include "st_surrogate.h"

namespace {

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// the outputs of the call under way, and what its launches said
struct Buffer { const char* p; size_t bytes; };
std::vector<Buffer> g_outputs;
int g_masked_grads = 0, g_masked_strided = 0, g_masked_layers = 0, g_angles = 0;
const uint8_t* g_tables[3] = {nullptr, nullptr, nullptr};  // y, z, grad of the last gradient launch
int64_t g_table_len = 0;
int g_reach = 0, g_wide_angles = 0, g_since_grad = 0;
bool g_any_output = false;  // outputs that the library allocates itself
std::vector<int> g_grad_pieces;  // z pieces of the gradient launches, chunk by chunk

bool inside_outputs(const void* p, size_t bytes) {
  if (g_any_output) return true;
  for (const Buffer& b : g_outputs)
    if (p >= b.p && static_cast<const char*>(p) + bytes <= b.p + b.bytes) return true;
  return false;
}

}  // namespace

namespace st {

#define ST_PAIR(ret, name, mangled, args)                   \
  ret real_##name args asm("__real_" mangled);              \
  ret wrap_##name args asm("__wrap_" mangled);
ST_PAIR(hipError_t, grad, "_ZN2st17launch_grad_fusedEiiRKNS_15GradFusedParamsEP12ihipStream_t",
        (int R, int in_dtype, const GradFusedParams& p, hipStream_t stream))
ST_PAIR(hipError_t, grouped, "_ZN2st25launch_grad_fused_groupedEiiiRKNS_14GradFusedGroupElP12ihipStream_t",
        (int R, int in_dtype, int rows, const GradFusedGroup& p, int64_t blocks, hipStream_t stream))
ST_PAIR(hipError_t, strided, "_ZN2st14launch_stridedEiibRKNS_13StridedParamsEP12ihipStream_t",
        (int R, int in_dtype, bool with_d, const StridedParams& p, hipStream_t stream))
ST_PAIR(hipError_t, conv, "_ZN2st14launch_sg_convEiiRKNS_12SgConvParamsEP12ihipStream_t",
        (int layer, int dtype, const SgConvParams& p, hipStream_t stream))
ST_PAIR(hipError_t, angles, "_ZN2st13launch_anglesERKNS_12AnglesParamsEP12ihipStream_t",
        (const AnglesParams& p, hipStream_t stream))
#undef ST_PAIR

hipError_t wrap_grad(int R, int in_dtype, const GradFusedParams& p, hipStream_t stream) {
  g_grad_pieces.push_back(p.nchunks);
  g_since_grad = 0;
  if (p.cells != nullptr) {
    ++g_masked_grads;
    const MaskCells& c = p.mask;
    const int64_t cz = cells_of(p.nz), cy = cells_of(p.ny), cx = cells_of(p.nx), xs = cdiv(p.nx, 64);
    const int64_t n = p.nz * p.ny * p.nx, table = cz * cy * xs;
    if (c.mask == nullptr) hc::violation("mask cells without a mask");
    hc::need(c.mask, static_cast<size_t>(n), "mask");
    const size_t bytes = static_cast<size_t>(mask_cell_bytes(p.nz, p.ny, p.nx));
    hc::need(c.base, bytes, "mask cells");
    if (!inside_outputs(c.base, bytes)) hc::violation("the mask cells do not lie in an output of the call");
    if (c.y != c.base + cz * cy * cx || c.z != c.y + table || c.grad != c.z + table ||
        c.grad + table != c.base + bytes)
      hc::violation("the cell tables overlap or leave their bytes");
    if (p.cells != c.grad) hc::violation("the gradient pass reads another table");
    if (p.x_tiles != xs || (p.rows != 4 && p.rows != 8)) hc::violation("cells of other tiles than the gradient's");
    g_tables[0] = c.y; g_tables[1] = c.z; g_tables[2] = c.grad;
    g_table_len = table;
    g_reach = c.reach;
  } else {
    g_tables[0] = g_tables[1] = g_tables[2] = nullptr;
  }
  return real_grad(R, in_dtype, p, stream);
}

hipError_t wrap_grouped(int R, int in_dtype, int rows, const GradFusedGroup& p, int64_t blocks, hipStream_t stream) {
  for (int e = 0; e < p.g.count; ++e) g_grad_pieces.push_back(p.g.geo[e].nchunks);
  return real_grouped(R, in_dtype, rows, p, blocks, stream);
}

hipError_t wrap_strided(int R, int in_dtype, bool with_d, const StridedParams& p, hipStream_t stream) {
  if (p.cells != nullptr) {
    ++g_masked_strided;
    const bool zaxis = g_since_grad++ == 0;  // z, then y
    if (with_d || in_dtype != ST_DTYPE_F32 || p.so_axis != p.s_axis || p.so_other != p.s_other)
      hc::violation("cells given to a pass that does without");
    if (p.cells != g_tables[zaxis ? 1 : 0]) hc::violation("the %c integration of %lld x %lld x %lld reads another table", zaxis ? 'z' : 'y', (long long)p.n_axis, (long long)p.n_other, (long long)p.nx);
    if (R != g_reach) hc::violation("cells dilated by %d for an integration of radius %d", g_reach, R);
    const int64_t xs = cdiv(p.nx, 64), cy = cells_of(zaxis ? p.n_other : p.n_axis);
    const int64_t za = cy * xs, ya = xs;  // strides of a cell along z and y
    if (p.cell_axis != (zaxis ? za : ya) || p.cell_other != (zaxis ? ya : za)) hc::violation("cell strides");
    const int64_t last = (cells_of(p.n_axis) - 1) * p.cell_axis + (cells_of(p.n_other) - 1) * p.cell_other + xs - 1;
    if (last + 1 != g_table_len) hc::violation("cell indices reach %lld of %lld", (long long)last, (long long)g_table_len);
  }
  return real_strided(R, in_dtype, with_d, p, stream);
}

hipError_t wrap_conv(int layer, int dtype, const SgConvParams& p, hipStream_t stream) {
  static bool built = false;
  if (layer == 1 && p.z_lo == 0) built = false;
  if ((p.cells != nullptr) != (p.work != nullptr)) hc::violation("cells without a work count");
  if (p.cells != nullptr) {
    ++g_masked_layers;
    if (p.mask == nullptr) hc::violation("cells without a mask");
    hc::need(p.mask, static_cast<size_t>(p.n), "mask");
    hc::need(p.cells, static_cast<size_t>(sg_cells(p.nz) * sg_cells(p.ny) * sg_cells(p.nx)), "surrogate mask cells");
    hc::need(p.work, sizeof(int), "surrogate work count");
    if (reinterpret_cast<uintptr_t>(p.work) % sizeof(int)) hc::violation("an unaligned work count");
    static int64_t seen = 0;  // planes that layer 1 has been launched over
    if (layer == 1) seen = p.z_lo == 0 ? p.z_hi : seen + p.z_hi - p.z_lo;
    if (p.work_planes != seen) hc::violation("work counted over %lld planes, not %lld", (long long)p.work_planes, (long long)seen);
    if (p.reach != kSgLayers - layer) hc::violation("layer %d reaches %d voxels", layer, p.reach);
    if (layer == 1 && p.build_cells) built = true;
    if (!built) hc::violation("layer %d reads cells that no launch made", layer);
  }
  return real_conv(layer, dtype, p, stream);
}

hipError_t wrap_angles(const AnglesParams& p, hipStream_t stream) {
  ++g_angles;
  if (p.n < 1 || p.n >= (int64_t(1) << 51) || cdiv(p.n, 1024) > INT32_MAX) hc::violation("k_angles: grid");
  g_wide_angles += p.vec_ok != 0;
  if (p.vec_ok) {  // a lane's four voxels in one access
    if (p.n % 4 != 0) hc::violation("k_angles: 16-byte accesses to planes of %lld", (long long)p.n);
    for (const void* q : {(const void*)p.e3, (const void*)p.ha, (const void*)p.ia})
      if (reinterpret_cast<uintptr_t>(q) % 16) hc::violation("k_angles: 16-byte accesses to an unaligned buffer");
    for (const void* q : {(const void*)p.mask, (const void*)p.flags})
      if (reinterpret_cast<uintptr_t>(q) % 4) hc::violation("k_angles: 4-byte accesses to an unaligned buffer");
  }
  return real_angles(p, stream);
}

}  // namespace st

namespace {

void expect(int got, int want, const char* what) {
  if (got != want) {
    std::fprintf(stderr, "plans FAIL: %s returned %d, expected %d (%s)\n", what, got, want, st_last_error());
    std::exit(1);
  }
}

void* dev(size_t bytes) {
  void* p = nullptr;
  if (hipMalloc(&p, bytes) != hipSuccess || p == nullptr) {
    std::fprintf(stderr, "plans FAIL: stub allocation of %zu bytes\n", bytes);
    std::exit(1);
  }
  return p;
}

const double kC[3] = {10.5, 11.25, 19.5}, kD[3] = {1.0, 0.2, -0.1};

// One masked st_compute with a caller workspace and the outputs whose letters are
// in `which` (e: e3, v: evals, f: fa, h: ha, i: ia, b: flags).
void masked_call(int64_t nz, int64_t ny, int64_t nx, double sigma, double rho, const char* which, bool mask = true) {
  const int64_t n = nz * ny * nx;
  void* vol = dev(static_cast<size_t>(n) * 2);
  uint8_t* m = mask ? static_cast<uint8_t*>(dev(static_cast<size_t>(n))) : nullptr;
  g_outputs.clear();
  auto out = [&](char k, size_t bytes) -> void* {
    if (std::strchr(which, k) == nullptr) return nullptr;
    void* p = dev(bytes);
    g_outputs.push_back(Buffer{static_cast<const char*>(p), bytes});
    return p;
  };
  const size_t N = static_cast<size_t>(n);
  float* e3 = static_cast<float*>(out('e', 12 * N));
  float* ev = static_cast<float*>(out('v', 12 * N));
  float* fa = static_cast<float*>(out('f', 4 * N));
  float* ha = static_cast<float*>(out('h', 4 * N));
  float* ia = static_cast<float*>(out('i', 4 * N));
  uint8_t* fl = static_cast<uint8_t*>(out('b', N));
  const size_t wsb = st_workspace_bytes(nz, ny, nx);
  void* ws = dev(wsb);
  expect(st_compute(vol, ST_DTYPE_U16, m, nz, ny, nx, sigma, rho, 4.0, kC, kD, e3, ev, fa, ha, ia, fl, ws, wsb,
                    nullptr),
         ST_OK, "st_compute");
  for (void* p : {vol, (void*)m, (void*)e3, (void*)ev, (void*)fa, (void*)ha, (void*)ia, (void*)fl, ws}) (void)hipFree(p);
}

// A mask's cells are made from 2^22 voxels on, for the fused gradient.
void threshold() {
  struct Case { int64_t nz, ny, nx; double sigma; bool mask; int cells; };
  for (const Case& c : {Case{127, 128, 256, 1.0, true, 0}, Case{128, 128, 256, 1.0, true, 1},
                        Case{128, 128, 256, 1.0, false, 0}, Case{128, 128, 256, 2.6, true, 0}}) {
    g_masked_grads = g_masked_strided = 0;
    masked_call(c.nz, c.ny, c.nx, c.sigma, 2.0, "b", c.mask);
    if (g_masked_grads != c.cells || g_masked_strided != 2 * c.cells)
      hc::violation("%lld x %lld x %lld, sigma %g: %d masked gradient launches, expected %d", (long long)c.nz,
                    (long long)c.ny, (long long)c.nx, c.sigma, g_masked_grads, c.cells);
  }
}

// One masked st_surrogate_infer in z slabs of `slab` planes; layers with cells.
int surrogate_call(int64_t nz, int64_t ny, int64_t nx, int64_t slab, double min_confidence) {
  const int64_t n = nz * ny * nx;
  const size_t N = static_cast<size_t>(n);
  setenv("ST_SURROGATE_SLAB_BYTES", std::to_string(2 * (slab + 8) * ny * nx * 64).c_str(), 1);
  void* vol = dev(2 * N);
  uint8_t* m = static_cast<uint8_t*>(dev(N));
  float* w = static_cast<float*>(dev(4 * ST_SURROGATE_WEIGHTS));
  float* fa = static_cast<float*>(dev(4 * N));
  g_masked_layers = 0;
  expect(st_surrogate_infer(vol, ST_DTYPE_U16, m, nz, ny, nx, w, 4 * ST_SURROGATE_WEIGHTS, min_confidence, 1.0, 2.0, 4.0,
                            kC, kD, nullptr, fa, nullptr, nullptr, nullptr, nullptr),
         ST_OK, "st_surrogate_infer");
  for (void* p : {vol, (void*)m, (void*)w, (void*)fa}) (void)hipFree(p);
  unsetenv("ST_SURROGATE_SLAB_BYTES");
  return g_masked_layers;
}

// The surrogate makes its own from 2^20 voxels on.
void surrogate_threshold() {
  if (surrogate_call(127, 64, 128, 32, 0.0) != 0) hc::violation("cells below 2^20 voxels");
  if (surrogate_call(128, 64, 128, 32, 0.0) != 4 * 5) hc::violation("no cells at 2^20 voxels in four slabs");
}

// z pieces of the gradient pass for a launch shape.
int pieces(int64_t nz, int64_t ny, int64_t nx, double sigma, const st::host::LaunchShape& shape) {
  static uint16_t vol[1];
  static float out[1];
  st::host::PathArgs a;
  expect(st::host::prepare_path(a, vol, ST_DTYPE_U16, nullptr, nz, ny, nx, sigma, 2.0, 4.0, nullptr, nullptr, nullptr,
                                nullptr, out, nullptr, nullptr, nullptr),
         ST_OK, "prepare_path");
  st::host::PathPlan plan;
  st::host::plan_path(a, reinterpret_cast<char*>(uintptr_t(1) << 32), shape, &plan);  // addresses only
  return plan.grad.nchunks;
}

// How far the gradient pass splits z: a target above the chip plans for the chip,
// and whether a launch has it for itself is said, not taken from the target.
void split() {
  const int64_t sizes[][3] = {{64, 64, 64}, {120, 90, 200}, {48, 300, 300}, {200, 40, 333}, {90, 512, 512}, {33, 65, 700}};
  int differ = 0;
  for (const auto& q : sizes)
    for (double sigma : {1.0, 1.5, 2.0}) {
      st::host::LaunchShape chip, more, beside;
      more.grad_min_blocks = 4 * chip.grad_min_blocks;
      beside.alone = false;
      const int n = pieces(q[0], q[1], q[2], sigma, chip);
      if (pieces(q[0], q[1], q[2], sigma, more) != n)
        hc::violation("%lld x %lld x %lld, sigma %g: %d pieces for four chips, %d for one", (long long)q[0],
                      (long long)q[1], (long long)q[2], sigma, pieces(q[0], q[1], q[2], sigma, more), n);
      differ += pieces(q[0], q[1], q[2], sigma, beside) != n;
    }
  if (differ == 0) hc::violation("a launch beside others is planned as one alone");
  // chains: two chunks in one chain have the chip one after the other, in two beside
  // each other; grouped: one chunk has it, two share it
  const int64_t N = 64 * 64 * 64;
  std::vector<st_chunk> chunks(2);
  for (st_chunk& c : chunks) {
    c = st_chunk{};
    c.volume = dev(2 * N); c.dtype = ST_DTYPE_U16;
    c.nz = c.ny = c.nx = 64; c.rho = 2.0;
    c.fa = static_cast<float*>(dev(4 * N));
  }
  auto batch_pieces = [&](int count, int lanes) {
    g_grad_pieces.clear();
    st_batch* b = nullptr;
    expect(st_batch_create(chunks.data(), count, 1.0, 4.0, nullptr, nullptr, lanes, nullptr, 0, &b), ST_OK,
           "st_batch_create");
    expect(st_batch_destroy(b), ST_OK, "st_batch_destroy");
    return g_grad_pieces;
  };
  st::host::LaunchShape chip, quarter, half;
  quarter.grad_min_blocks = chip.grad_min_blocks / 4;
  half.grad_min_blocks = chip.grad_min_blocks / 2;
  quarter.alone = half.alone = false;
  const std::vector<int> one(2, pieces(64, 64, 64, 1.0, chip)), two(2, pieces(64, 64, 64, 1.0, quarter));
  if (batch_pieces(2, 1) != one) hc::violation("one chain: not planned as alone");
  if (batch_pieces(2, 2) != two) hc::violation("two chains: planned otherwise than beside each other");
  if (batch_pieces(1, ST_BATCH_GROUPED) != std::vector<int>(1, one[0])) hc::violation("a grouped round of one chunk");
  if (batch_pieces(2, ST_BATCH_GROUPED) != std::vector<int>(2, pieces(64, 64, 64, 1.0, half)))
    hc::violation("a grouped round of two chunks");
  for (st_chunk& c : chunks) {
    (void)hipFree(const_cast<void*>(c.volume));
    (void)hipFree(c.fa);
  }
}

// Where the cells of masked calls lie: in the first output asked for, whichever that
// is and however few bytes it has (flags: one a voxel), for thin shapes and sizes on
// and off the cells' edges, or nowhere if they would not fit; of a chunk batch's
// chunks each in its own outputs; of the surrogate's in its own scratch, in slabs and
// with the whole-volume fallback.
void cells() {
  const int64_t sizes[][3] = {{128, 256, 256}, {129, 251, 263}, {9, 1000, 1000}, {1000, 1000, 9}, {65, 8, 17000}};
  for (const auto& q : sizes)
    for (const char* which : {"b", "f", "vb"}) {
      g_masked_grads = g_masked_strided = 0;
      masked_call(q[0], q[1], q[2], 1.0, 2.0, which);
      if (g_masked_grads != 1 || g_masked_strided != 2) hc::violation("a masked call without cells");
    }
  masked_call(int64_t(1) << 23, 1, 1, 1.0, 2.0, "b");  // a column: half a byte of cells a voxel
  // chains and grouped rounds
  const int64_t nz = 128, ny = 256, nx = 257, N = nz * ny * nx;
  std::vector<st_chunk> chunks(3);
  g_outputs.clear();
  for (size_t i = 0; i < chunks.size(); ++i) {
    st_chunk& c = chunks[i];
    c = st_chunk{};
    c.volume = dev(2 * N); c.dtype = ST_DTYPE_U16;
    if (i != 1) c.mask = static_cast<uint8_t*>(dev(N));
    c.nz = nz; c.ny = ny; c.nx = nx; c.rho = 2.0;
    c.flags = static_cast<uint8_t*>(dev(N));
    g_outputs.push_back(Buffer{reinterpret_cast<const char*>(c.flags), static_cast<size_t>(N)});
  }
  for (int lanes : {1, 2, ST_BATCH_GROUPED}) {
    g_masked_grads = 0;
    const size_t wsb = st_batch_workspace_bytes(chunks.data(), 3, lanes == ST_BATCH_GROUPED ? 1 : lanes);
    void* ws = dev(wsb);
    st_batch* b = nullptr;
    expect(st_batch_create(chunks.data(), 3, 1.0, 4.0, nullptr, nullptr, lanes, ws, wsb, &b), ST_OK, "st_batch_create");
    int kernels = 0;
    expect(st_batch_plan(b, nullptr, nullptr, &kernels), ST_OK, "st_batch_plan");
    const bool chains = lanes != ST_BATCH_GROUPED;
    if (g_masked_grads != (chains ? 2 : 0)) hc::violation("%d chunks with cells", g_masked_grads);
    if (chains && kernels != 3 * 4 + 2 * 2) hc::violation("a plan of %d kernels", kernels);
    expect(st_batch_launch(b, nullptr), ST_OK, "st_batch_launch");
    expect(st_batch_destroy(b), ST_OK, "st_batch_destroy");
    (void)hipFree(ws);
  }
  for (st_chunk& c : chunks) {
    (void)hipFree(const_cast<void*>(c.volume));
    (void)hipFree(const_cast<uint8_t*>(c.mask));
    (void)hipFree(c.flags);
  }
  // the surrogate
  if (surrogate_call(129, 251, 263, 40, 0.0) != 4 * 5) hc::violation("layers without cells");
  setenv("HOSTCHECK_FLAGS", "all", 1);
  g_outputs.clear();
  g_any_output = true;  // the fallback's temporaries
  if (surrogate_call(129, 251, 263, 40, 0.9) != 4 * 5) hc::violation("layers without cells (fallback)");
  g_any_output = false;
  unsetenv("HOSTCHECK_FLAGS");
}

// The re-angling call: 16-byte accesses only where every buffer and plane allows.
void angles() {
  for (int64_t nx : {64, 65, 66, 68, 1})
    for (int shift : {0, 1, 2, 4}) {  // floats past a 16-byte start, bytes past a 4-byte one
      const int64_t nz = 3, ny = 5, n = nz * ny * nx;
      float* e3 = static_cast<float*>(dev(4 * (3 * n + 8)));
      float* ha = static_cast<float*>(dev(4 * (n + 8)));
      uint8_t* bytes = static_cast<uint8_t*>(dev(2 * n + 16));
      for (int which = 0; which < 5; ++which) {
        const int a = which == 0 ? shift : 0, b = which == 1 ? shift : 0, m = which == 2 ? shift : 0,
                  f = which == 3 ? shift : 0;
        expect(st_angles(e3 + a, bytes + m, nz, ny, nx, kC, kD, ha + b, nullptr, bytes + n + 8 - (n + 8) % 4 + f, nullptr),
               ST_OK, "st_angles");
      }
      (void)hipFree(e3);
      (void)hipFree(ha);
      (void)hipFree(bytes);
    }
  if (g_angles != 5 * 4 * 5) hc::violation("%d re-angling launches", g_angles);
  if (g_wide_angles == 0 || g_wide_angles == g_angles) hc::violation("%d of them wide", g_wide_angles);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "threshold") threshold();
  else if (what == "surrogate_threshold") surrogate_threshold();
  else if (what == "split") split();
  else if (what == "cells") cells();
  else if (what == "angles") angles();
  else return 2;
  if (hc::live_objects() != 0) {
    std::printf("plans: FAIL (objects leaked)\n");
    return 1;
  }
  std::printf("plans: OK\n");
  return 0;
}
