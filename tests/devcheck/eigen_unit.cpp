// e3 comes out of the solution as a unit vector in float64: its length is 1 to a
// few roundings (2^-50), however coarse the reciprocal square root's estimate
// was, for tensors of many sizes, shapes and directions.
#include "devcheck.h"

#include <random>

#include "st_device.h"

unsigned __lane_id() { return 0; }
unsigned long long __ballot(int) { return 0; }

int main() {
  std::mt19937_64 gen(7);
  std::normal_distribution<double> normal;
  double worst = 0.0;
  for (int i = 0; i < 200000; ++i) {
    // a sum of three rank-one tensors of decreasing weight, at any scale
    double t[6] = {0, 0, 0, 0, 0, 0};
    const double scale = std::pow(10.0, i % 25 - 12);
    for (int k = 0; k < 3; ++k) {
      const double g[3] = {normal(gen), normal(gen), normal(gen)}, w = scale * std::pow(0.2, k);
      t[0] += w * g[0] * g[0]; t[1] += w * g[0] * g[1]; t[2] += w * g[0] * g[2];
      t[3] += w * g[1] * g[1]; t[4] += w * g[1] * g[2]; t[5] += w * g[2] * g[2];
    }
    st::EigOut o;
    st::eig_smallest(t, true, o);
    const double len = std::sqrt(static_cast<double>(o.vz) * o.vz + static_cast<double>(o.vy) * o.vy +
                                 static_cast<double>(o.vx) * o.vx);
    worst = std::fmax(worst, std::fabs(len - 1.0));
  }
  if (!(worst <= 0x1p-50)) {
    std::printf("largest deviation of |e3| from 1: %g\n", worst);
    dc::fail("e3 is not of unit length in float64");
  }
  std::printf("devcheck: OK (%g)\n", worst);
}
