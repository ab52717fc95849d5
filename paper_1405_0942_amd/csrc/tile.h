// tile.h -- the points of a z-marching tile (stage.hip): which point of the stage-input window (tile and
// 2-node halo) and of the field window (1-node halo) a thread has, and where the sweep reads the stage
// input for it.  Plain integer code that the host can run too.  Internal to the library.
#pragma once

#include "relax_device.h"

namespace relax {

// Which axes of a grid may be line-tied in a marching kernel: none, z alone, any
enum { FACES_NONE = 0, FACES_Z = 1, FACES_XY = 2 };
inline int faces_of(const Geometry& g) {
  if (g.bc[0] == BC_LINE_TIED || g.bc[1] == BC_LINE_TIED) return FACES_XY;
  return g.bc[2] == BC_LINE_TIED ? FACES_Z : FACES_NONE;
}

struct TilePoint {
  int row, col;  // in its window
};

// Both windows: point e < tw th is the tile node of thread e, so that each thread has its own node.
// div(e, d): e / d.  Stage-input window, then the two rows below and the two above the tile, then the two
// columns on either side
template <typename Div>
__host__ __device__ __forceinline__ TilePoint window_point(int e, int tw, int th, Div div) {
  const int wx2 = tw + 4, wy2 = th + 4;
  TilePoint p;
  if (e < tw * th) {
    p.row = div(e, tw) + 2;
    p.col = e - (p.row - 2) * tw + 2;
  } else {
    const int e2 = e - tw * th;
    if (e2 < 4 * wx2) {
      const int band = div(e2, wx2);
      p.row = band < 2 ? band : wy2 - 4 + band;
      p.col = e2 - band * wx2;
    } else {
      const int e3 = e2 - 4 * wx2, side = e3 & 3;
      p.row = 2 + (e3 >> 2);
      p.col = side < 2 ? side : wx2 - 4 + side;
    }
  }
  return p;
}

// Field window, then the ring around the tile
template <typename Div>
__host__ __device__ __forceinline__ TilePoint field_point(int e, int tw, int th, Div div) {
  const int wx1 = tw + 2, wy1 = th + 2;
  TilePoint p;
  if (e < tw * th) {
    p.row = div(e, tw) + 1;
    p.col = e - (p.row - 1) * tw + 1;
  } else {
    const int e2 = e - tw * th;
    if (e2 < wx1) {
      p.row = 0;
      p.col = e2;
    } else if (e2 < 2 * wx1) {
      p.row = wy1 - 1;
      p.col = e2 - wx1;
    } else {
      const int e3 = e2 - 2 * wx1;
      p.row = 1 + (e3 >> 1);
      p.col = (e3 & 1) ? wx1 - 1 : 0;
    }
  }
  return p;
}

// Offset of field point p in the stage-input window.  A tile of fewer than 512 field points has threads
// past the window that evaluate a point all the same (nothing of it is kept): those take the tile's first
// node, whose neighbours lie in the window as well.
__host__ __device__ __forceinline__ int field_offset(TilePoint p, bool in_window, int tw) {
  const int wx2 = tw + 4;
  return in_window ? (p.row + 1) * wx2 + p.col + 1 : 2 * wx2 + 2;
}

// The two points (plus | minus << 16) whose difference is F' along an axis at offset o of the stage-input window,
// s a step along it: its neighbours; on a line-tied face (end 1: low, 2: high) the sum 4 y(1) - 3 y(0), which
// stands beyond it, and y(2)
__host__ __device__ __forceinline__ int difference_points(int o, int s, int end) {
  const int plus = end == 1 ? o - s : (end == 2 ? o - 2 * s : o + s);
  const int minus = end == 1 ? o + 2 * s : (end == 2 ? o + s : o - s);
  return plus | minus << 16;
}

}  // namespace relax
