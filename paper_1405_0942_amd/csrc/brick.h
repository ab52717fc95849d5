// brick.h -- the points of a brick (small-grid sweeps: brick.hip and the reverse sweeps of
// adjoint.hip): strides of its windows, and which grid node and wrap a window point or a field
// point is.  Internal to the library.
#pragma once

#include "sweep_common.h"

namespace relax {

// The value at element i of a component, i < 2^28: base in scalar registers, byte offset in one register
template <typename V>
__device__ __forceinline__ V at(const V* __restrict__ base, unsigned i) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + i * (unsigned)sizeof(V));
}

struct Brick {
  int bx, by, bz;    // nodes
  int sx, sy, sxy;   // strides of the stage-input window (2-node halo)
  int fx, fxy;       // strides of the field window (1-node halo)
  int nwin, nown, nshell;  // points of the window, nodes, field points around them
  __device__ __forceinline__ explicit Brick(const Geometry& g)
      : bx(g.brick[0]), by(g.brick[1]), bz(g.brick[2]), sx(bx + 4), sy(by + 4), sxy(sx * sy), fx(bx + 2),
        fxy(fx * (by + 2)), nwin(sxy * (bz + 4)), nown(bx * by * bz),
        nshell(fxy * (bz + 2) - nown) {}
  // whether the window of the brick at (i0, j0, k0) reaches beyond a line-tied face
  __device__ __forceinline__ bool at_face(const Geometry& g, int i0, int j0, int k0) const {
    return (g.bc[0] == BC_LINE_TIED && (i0 <= 1 || i0 + bx >= g.n[0] - 1)) ||
           (g.bc[1] == BC_LINE_TIED && (j0 <= 1 || j0 + by >= g.n[1] - 1)) ||
           (g.bc[2] == BC_LINE_TIED && (k0 <= 1 || k0 + bz >= g.n[2] - 1));
  }
};

// Where the brick of this workgroup begins
struct BrickOrigin {
  int i0, j0, k0;
  __device__ __forceinline__ BrickOrigin(const Brick& b, const Geometry& g) {
    const int lb = logical_block(blockIdx.x, g.nblocks);
    const int row = __builtin_amdgcn_readfirstlane(small_div(lb, g.tiles[0]));
    const int plane = __builtin_amdgcn_readfirstlane(small_div(row, g.tiles[1]));
    i0 = (lb - row * g.tiles[0]) * b.bx;
    j0 = (row - plane * g.tiles[1]) * b.by;
    k0 = plane * b.bz;
  }
};

struct BrickPoint {
  int index;  // grid index (0 off the grid)
  int wraps;  // periodic wraps of x, y, z, each + 1, in bits 0-1, 2-3, 4-5; bit 6: on the grid
  __device__ __forceinline__ bool on() const { return wraps & 64; }
  __device__ __forceinline__ double wrap(int m) const { return (double)(((wraps >> (2 * m)) & 3) - 1); }
};

// window point e < nwin
__device__ __forceinline__ BrickPoint brick_window(const Brick& b, const Geometry& g, int e, const BrickOrigin& at) {
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int lz = small_div(e, b.sxy), e2 = e - __mul24(lz, b.sxy), ly = small_div(e2, b.sx), lx = e2 - __mul24(ly, b.sx);
  const AxisIdx rx = axis_index(at.i0 + lx - 2, nx, g.bc[0]), ry = axis_index(at.j0 + ly - 2, ny, g.bc[1]);
  const AxisIdx rz = axis_index(at.k0 + lz - 2, nz, g.bc[2]);
  BrickPoint p;
  const bool on = rx.ok && ry.ok && rz.ok;
  p.index = on ? __mul24(__mul24(rz.i, ny) + ry.i, nx) + rx.i : 0;
  p.wraps = (rx.w + 1) | (ry.w + 1) << 2 | (rz.w + 1) << 4 | (on ? 64 : 0);
  return p;
}

struct BrickField {
  int index;   // grid index (0 where !ok)
  int slot;    // offset in the field window, -1: no point
  int window;  // offset in the stage-input window
  int ends;    // line-tied ends it lies on: 1, 2 along x, 4, 8 along y, 16, 32 along z; 64: on the
               // grid (on periodic axes also where the brick overhangs it); 128: r = 0, a node of the brick
  __device__ __forceinline__ bool on() const { return ends & 64; }
  __device__ __forceinline__ bool node() const { return ends & 128; }
  __device__ __forceinline__ bool face() const { return ends & 63; }
};

// field point r of thread tid: r = 0 is the own node; then the shell: the planes below and above the
// brick, then a ring around each of its planes
__device__ __forceinline__ BrickField brick_field(const Brick& b, const Geometry& g, int r, int tid, const BrickOrigin& at) {
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  int cx, cy, cz;  // field window coordinates
  bool in;
  if (r == 0) {
    in = tid < b.nown;
    const int e = in ? tid : 0, bxy = __mul24(b.bx, b.by);
    const int tz = small_div(e, bxy), e2 = e - __mul24(tz, bxy), ty = small_div(e2, b.bx);
    cx = e2 - __mul24(ty, b.bx) + 1;
    cy = ty + 1;
    cz = tz + 1;
  } else {
    const int e = tid + (r - 1) * BRICK_THREADS, ring = 2 * (b.fx + b.by);
    if (e < 2 * b.fxy) {
      const int top = e >= b.fxy ? 1 : 0, e2 = e - (top ? b.fxy : 0);
      cz = top ? b.bz + 1 : 0;
      cy = small_div(e2, b.fx);
      cx = e2 - __mul24(cy, b.fx);
      in = true;
    } else {
      const int e2 = e - 2 * b.fxy, layer = small_div(e2, ring), e3 = e2 - __mul24(layer, ring);
      in = layer < b.bz;
      cz = in ? layer + 1 : 0;
      if (e3 < 2 * b.fx) {
        cy = e3 < b.fx ? 0 : b.by + 1;
        cx = e3 < b.fx ? e3 : e3 - b.fx;
      } else {
        cy = 1 + ((e3 - 2 * b.fx) >> 1);
        cx = (e3 & 1) ? b.bx + 1 : 0;
      }
    }
  }
  const AxisIdx rx = axis_index(at.i0 + cx - 1, nx, g.bc[0]), ry = axis_index(at.j0 + cy - 1, ny, g.bc[1]);
  const AxisIdx rz = axis_index(at.k0 + cz - 1, nz, g.bc[2]);
  BrickField p;
  const bool on = in && rx.ok && ry.ok && rz.ok;
  p.slot = in ? __mul24(cz, b.fxy) + __mul24(cy, b.fx) + cx : -1;
  p.window = __mul24(cz + 1, b.sxy) + __mul24(cy + 1, b.sx) + cx + 1;
  p.ends = on ? 64 : 0;
  if (r == 0 && in && at.i0 + cx - 1 < nx && at.j0 + cy - 1 < ny && at.k0 + cz - 1 < nz) p.ends |= 128;
  if (g.bc[0] == BC_LINE_TIED) p.ends |= rx.i == 0 ? 1 : (rx.i == nx - 1 ? 2 : 0);
  if (g.bc[1] == BC_LINE_TIED) p.ends |= ry.i == 0 ? 4 : (ry.i == ny - 1 ? 8 : 0);
  if (g.bc[2] == BC_LINE_TIED) p.ends |= rz.i == 0 ? 16 : (rz.i == nz - 1 ? 32 : 0);
  p.index = on ? __mul24(__mul24(rz.i, ny) + ry.i, nx) + rx.i : 0;
  return p;
}

// F' at the field point with offset o in the window: central differences, on line-tied faces the one-sided
// rows, formed here by the few points that need them: a pass that wrote them to LDS took a barrier more (us per
// step, 33^3 49.9 -> 45.6, 65^3 107 -> 97).
template <typename Y>
__device__ __forceinline__ void face_differences(const Brick& b, int ends, bool at_face, const Y& ys, int o, double F[3][3]) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    const int s = c == 0 ? 1 : (c == 1 ? b.sx : b.sxy);
    double lo[3], hi[3];
#pragma unroll
    for (int m = 0; m < 3; m++) {
      lo[m] = ys[m][o - s];
      hi[m] = ys[m][o + s];
    }
    if (at_face) {
      const int end = (ends >> (2 * c)) & 3;  // 1: low end, 2: high end
      if (end == 1) {
#pragma unroll
        for (int m = 0; m < 3; m++) {
          hi[m] = face_sum(ys[m][o], hi[m]);
          lo[m] = ys[m][o + 2 * s];
        }
      } else if (end == 2) {
#pragma unroll
        for (int m = 0; m < 3; m++) {
          lo[m] = face_sum(ys[m][o], lo[m]);
          hi[m] = ys[m][o - 2 * s];
        }
      }
    }
#pragma unroll
    for (int m = 0; m < 3; m++) F[m][c] = hi[m] - lo[m];
  }
}

}  // namespace relax
