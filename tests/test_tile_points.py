"""Where a fitted tile of the z-march reads its window in LDS (tile.h), for every thread, on the CPU: also
the threads past a field window of fewer points than threads read inside the plane's window."""
import host_check

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <utility>
#include "tile.h"
using namespace relax;

static int div_(int e, int d) { return e / d; }

// the tile of an n[0] x n[1] x n[2] grid, every thread and pass of stage_kernel
static int check(int tw, int th) {
  const int wx2 = tw + 4, wy2 = th + 4, wx1 = tw + 2, wy1 = th + 2;
  if (tw < 1 || th < 1 || tw * th > NTHREADS || wx2 * wy2 > RX2 * RY2 || wx1 * wy1 > RX1 * RY1) return 1;
  std::set<int> win, fld;
  for (int e = 0; e < 2 * NTHREADS; e++) {
    if (e < wx2 * wy2) {
      const TilePoint p = window_point(e, tw, th, div_);
      if (p.row < 0 || p.row >= wy2 || p.col < 0 || p.col >= wx2 || !win.insert(p.row * wx2 + p.col).second) return 2;
    }
    const TilePoint p = field_point(e, tw, th, div_);
    const bool in = e < wx1 * wy1;
    if (in && (p.row < 0 || p.row >= wy1 || p.col < 0 || p.col >= wx1 || !fld.insert(p.row * wx1 + p.col).second)) return 3;
    // a thread's own pass runs for all of them, the second for points of the window alone
    if (e < NTHREADS || in) {
      const int o = field_offset(p, in, tw);
      for (int s : {1, wx2})
        if (o - s < 0 || o + s >= wx2 * wy2) return 4;
      if (in && o != (p.row + 1) * wx2 + p.col + 1) return 5;
      // the points of F': a low face beyond column 0 is one of the columns 1 to tw, a high face likewise
      for (int end = 0; end < 3; end++)
        for (int axis = 0; axis < 2; axis++) {
          const int at = axis ? p.row : p.col, last = axis ? th : tw, s = axis ? wx2 : 1;
          if (in && end && (at < 1 || at > last)) continue;
          const int d = difference_points(o, s, end), plus = d & 0xffff, minus = d >> 16;
          if (plus >= wx2 * wy2 || minus < 0 || minus >= wx2 * wy2) return 7;
          if (plus != (end == 1 ? o - s : end == 2 ? o - 2 * s : o + s)) return 8;
          if (minus != (end == 1 ? o + 2 * s : end == 2 ? o + s : o - s)) return 8;
        }
    }
  }
  return (int)win.size() == wx2 * wy2 && (int)fld.size() == wx1 * wy1 ? 0 : 6;
}

int main() {
  std::set<std::pair<int, int>> tiles;
  auto take = [&](int nx, int ny, int nz) {
    for (int curl = 0; curl < 2; curl++) {
      relax_config c;
      std::memset(&c, 0, sizeof c);
      c.n[0] = nx;
      c.n[1] = ny;
      c.n[2] = nz;
      c.h[0] = c.h[1] = c.h[2] = 0.1;
      c.curl = curl;
      const Geometry g = make_geometry(&c);
      if (!g.brick[0]) tiles.insert({g.tw, g.th});
    }
  };
  take(67, 67, 203);
  take(129, 5, 900);
  take(130, 4, 1100);
  take(129, 129, 129);
  std::srand(1);
  for (int i = 0; i < 4000; i++) take(4 + std::rand() % 400, 4 + std::rand() % (i % 2 ? 400 : 24), 4 + std::rand() % 1200);
  int few = 0;
  for (auto t : tiles) {
    few += (t.first + 2) * (t.second + 2) < NTHREADS;
    if (int rc = check(t.first, t.second)) {
      std::printf("tile %d x %d: failure %d\n", t.first, t.second, rc);
      return 1;
    }
  }
  std::printf("%zu %d\n", tiles.size(), few);
  return 0;
}
"""


def test_every_read_of_a_fitted_tile_lies_in_its_window(tmp_path):
    tiles, few = map(int, host_check.run(SOURCE, tmp_path).split())
    assert tiles > 100 and few > 10  # `few`: fewer field points than threads
