// The runs of marked cells that a wave walks along an axis.  Against a walk written
// out here: every marked position of the piece lies in exactly one run, runs come in
// order and inside the piece; a gap of one or two cells between marked ones is part
// of a run, and of a longer gap no cell is (64 cells are looked at together, so a
// gap at the end of such a look stays open).  Gaps of every length, pieces that
// start and end inside a cell, axes of more than one look, random cells.
#include "devcheck.h"

#include "wave.h"

#include <algorithm>
#include <random>

#include "st_device.h"

struct Run { int a, len; };

std::vector<Run> walk(const std::vector<uint8_t>& cells, int stride, int a, int len) {
  std::vector<Run> runs;
  dc::run_wave([&] {
    st::CellRuns r(cells.data(), stride, a, len);
    int ra, rlen;
    while (r.next(ra, rlen))
      if (__lane_id() == 0) runs.push_back(Run{ra, rlen});
  });
  return runs;
}

void check(const std::vector<uint8_t>& marked, int stride, int a, int len) {
  std::vector<uint8_t> cells(marked.size() * stride, 0);
  for (size_t i = 0; i < marked.size(); ++i) cells[i * stride] = marked[i];
  const int first = a / 8, last = (a + len - 1) / 8;
  // expected cover, cell by cell of the piece
  std::vector<uint8_t> want(last + 1, 0);
  for (int look = first; look <= last; look += 64) {
    const int end = std::min(last + 1, look + 64);
    for (int c = look; c < end; ++c) {
      if (!marked[c]) continue;
      want[c] = 1;
      int next = c + 1;
      while (next < end && !marked[next]) ++next;
      if (next < end && next - c - 1 <= 2) std::fill(want.begin() + c, want.begin() + next, 1);
    }
  }
  std::vector<Run> expected;
  for (int c = first; c <= last; ++c) {
    if (!want[c]) continue;
    const int look_end = std::min(last + 1, first + (c - first) / 64 * 64 + 64);
    int e = c;
    while (e < look_end && want[e]) ++e;
    const int ra = std::max(8 * c, a), re = std::min(8 * e, a + len);
    expected.push_back(Run{ra, re - ra});
    c = e - 1;
  }
  const std::vector<Run> got = walk(cells, stride, a, len);
  bool same = got.size() == expected.size();
  for (size_t i = 0; same && i < got.size(); ++i) same = got[i].a == expected[i].a && got[i].len == expected[i].len;
  if (!same) {
    std::printf("piece [%d, %d), cells", a, a + len);
    for (int c = first; c <= last && c < first + 80; ++c) std::printf(" %d", marked[c]);
    std::printf("\n got");
    for (const Run& r : got) std::printf(" [%d, %d)", r.a, r.a + r.len);
    std::printf("\n expected");
    for (const Run& r : expected) std::printf(" [%d, %d)", r.a, r.a + r.len);
    std::printf("\n");
    dc::fail("runs of marked cells");
  }
}

int main() {
  for (int gap = 1; gap <= 8; ++gap) {  // two marked cells that far apart, at several places
    for (int at : {0, 5, 60, 63, 64}) {
      std::vector<uint8_t> m(90, 0);
      m[at] = m[at + gap + 1] = 1;
      check(m, 1, 0, 720);
      check(m, 3, 8 * at + 3, std::min(720 - 8 * at - 3, 8 * (gap + 2) - 5));
    }
  }
  std::mt19937 gen(3);
  for (int i = 0; i < 120; ++i) {
    const int n = 1 + static_cast<int>(gen() % 180);
    std::vector<uint8_t> m(n);
    const unsigned density = 1 + gen() % 8;
    for (uint8_t& c : m) c = gen() % 9 < density;
    const int a = static_cast<int>(gen() % (8 * n)), len = 1 + static_cast<int>(gen() % (8 * n - a));
    check(m, 1 + static_cast<int>(gen() % 4), a, len);
  }
  std::vector<uint8_t> all(150, 1);
  check(all, 1, 0, 1200);
  check(all, 1, 513, 600);
  std::printf("devcheck: OK\n");
}
