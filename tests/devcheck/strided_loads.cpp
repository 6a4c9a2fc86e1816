// A piece of an integration pass reads every sample of its window once: len outputs
// take len + 2 R loads a lane, whatever len is against the 2 R + 1 samples of the
// register window (fewer, a whole number of windows, one more), with nothing read
// again past the piece's end, and gives the filter's sums.  One lane of the
// kernel's own block runs here; its loads are counted.
#include "devcheck.h"

#include <algorithm>
#include <vector>

// what the block reads of a launch, and the loads and stores it makes
struct Index3 { unsigned x, y, z; };
static Index3 threadIdx, blockIdx;
static long g_loads = 0, g_stores = 0;
template <class T> T __builtin_nontemporal_load(const T* p) { ++g_loads; return *p; }
template <class T> void __builtin_nontemporal_store(T v, T* p) { ++g_stores; *p = v; }

#include "k_strided_impl.h"

unsigned __lane_id() { return 0; }
unsigned long long __ballot(int) { return 0; }

template <int R>
void check(int n, int pieces) {
  constexpr int W = 2 * R + 1;
  std::vector<float> in(n), out(n, -1.f);
  for (int i = 0; i < n; ++i) in[i] = static_cast<float>((i * 2654435761u >> 8) % 1000) / 7.f;
  st::Taps w;
  for (int k = 0; k < W; ++k) w.w[k] = 1.0 / (1.0 + std::abs(k - R));
  st::StridedGeo p{};
  p.job[0] = st::StridedJob{in.data(), out.data(), nullptr};
  p.njobs = 1;
  p.n_axis = n; p.s_axis = 1; p.so_axis = 1; p.n_other = 1; p.s_other = n; p.so_other = n;
  p.nx = 1; p.x_tiles = 1; p.o_tiles = 1;
  p.chunk = (n + pieces - 1) / pieces;
  p.nchunks = static_cast<int>((n + p.chunk - 1) / p.chunk);
  for (int c = 0; c < p.nchunks; ++c) {
    const int a = static_cast<int>(c * p.chunk), len = std::min<int>(n - a, static_cast<int>(p.chunk));
    g_loads = g_stores = 0;
    st::strided_impl::strided_block<R, float, false, true>(p, w, w, c);
    // a piece shorter than the window fills it all the same
    const long most = std::max(len, W) + 2 * R;
    if (g_loads > most || g_stores != len) {
      std::printf("R %d, piece of %d: %ld loads (at most %ld), %ld stores\n", R, len, g_loads, most, g_stores);
      dc::fail("loads of a piece");
    }
  }
  for (int i = 0; i < n; ++i) {
    double g = 0.0;
    for (int k = 0; k < W; ++k) g = std::fma(w.w[k], static_cast<double>(in[st::reflect_lane(i - R + k, n)]), g);
    if (static_cast<float>(g) != out[i]) dc::fail("an output of the pass");
  }
}

template <int R>
void radius() {
  constexpr int W = 2 * R + 1;
  for (int n : {1, 2, W - 1, W, W + 1, W + 3, 2 * W - 1, 2 * W, 2 * W + 1, 3 * W - 1, 3 * W, 5 * W + W / 2})
    for (int pieces : {1, 2, 3}) check<R>(n, pieces);
}

int main() {
  radius<1>();
  radius<4>();
  radius<16>();
  radius<32>();
  std::printf("devcheck: OK\n");
}
