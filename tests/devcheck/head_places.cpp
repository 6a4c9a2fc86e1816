// The training head's products read the LDS rows of 64 voxels, those of the wave
// itself: no place they read is in a row that another wave writes, and the places of
// the unused product rows are never written after they were cleared.
#include "devcheck.h"

typedef unsigned short __bf16;  // activations are not touched here

#include "st_surrogate.h"

unsigned __lane_id() { return 0; }
unsigned long long __ballot(int) { return 0; }

int main() {
  const int quantities = 11, product_rows = 16, voxels = 256;
  for (int wave = 0; wave < voxels / 64; ++wave)
    for (int row = 64 * wave; row < 64 * wave + 64; ++row)
      for (int q = 0; q < product_rows; ++q) {
        const int at = st::sg_head_place(row, q);
        if (at < 64 * wave * st::kSgHeadRow || at >= 64 * (wave + 1) * st::kSgHeadRow)
          dc::fail("a place in another wave's rows");
        for (int w = 0; w < quantities; ++w)
          if (q >= quantities && at == st::sg_head_place(row, w)) dc::fail("an unused product row reads a quantity");
        if (q < quantities && at != row * st::kSgHeadRow + q) dc::fail("the place of a quantity");
      }
  std::printf("devcheck: OK\n");
}
