// Two equal smaller eigenvalues (a volume that varies along one axis): e3 may be
// any vector of their plane, and is the first of the three cross products of rows
// 0 x 1, 0 x 2 and 1 x 2 of D - mu I that no other exceeds in length: along x where
// the tensor lies along z or y, along y where it lies along x (or the default
// (1, 0, 0) where all three vanish, with an eigenvalue that is exact).
#include "devcheck.h"

#include "st_device.h"

unsigned __lane_id() { return 0; }
unsigned long long __ballot(int) { return 0; }

int main() {
  int solved = 0;
  for (int axis = 0; axis < 3; ++axis)
    for (int i = 1; i <= 2000; ++i) {
      const double s = 0.37 * i * std::pow(10.0, i % 7 - 3);
      double t[6] = {0, 0, 0, 0, 0, 0};
      t[axis == 0 ? 0 : axis == 1 ? 3 : 5] = s;
      st::EigOut o;
      st::eig_smallest(t, true, o);
      if (!o.degenerate) dc::fail("a double eigenvalue is not flagged degenerate");
      const double want[3] = {0.0, axis == 2 ? 1.0 : 0.0, axis == 2 ? 0.0 : 1.0};
      if (o.vz == 1.0 && o.vy == 0.0 && o.vx == 0.0) continue;
      ++solved;
      if (!(std::fabs(o.vz - want[0]) < 1e-6 && std::fabs(o.vy - want[1]) < 1e-6 && std::fabs(o.vx - want[2]) < 1e-6)) {
        std::printf("axis %d scale %g: e3 = (%g, %g, %g)\n", axis, s, static_cast<double>(o.vz),
                    static_cast<double>(o.vy), static_cast<double>(o.vx));
        dc::fail("the tie between equal cross products");
      }
    }
  if (solved < 3000) dc::fail("too few tensors with an inexact eigenvalue");
  std::printf("devcheck: OK (%d)\n", solved);
}
