// brick.h -- the points of a brick (small-grid sweeps: brick.hip and the reverse sweeps of
// adjoint.hip): strides of its windows, and which grid node, wrap or ghost a window point or a field
// point is.  Internal to the library.
#pragma once

#include "sweep_common.h"

namespace relax {

// e / d for 0 <= e < 4096, 1 <= d < 4096: (e + 1/2) / d is at least 1 / (2 d) away from an integer,
// far more than the rounding of the reciprocal
__device__ __forceinline__ int small_div(int e, int d) {
  return (int)(((float)e + 0.5f) * __builtin_amdgcn_rcpf((float)d));
}

struct Brick {
  int bx, by, bz;    // nodes
  int sx, sy, sxy;   // strides of the stage-input window (2-node halo)
  int fx, fxy;       // strides of the field window (1-node halo)
  int nwin, nown;    // points of the window, nodes
  __device__ __forceinline__ explicit Brick(const Geometry& g)
      : bx(g.brick[0]), by(g.brick[1]), bz(g.brick[2]), sx(bx + 4), sy(by + 4), sxy(sx * sy), fx(bx + 2),
        fxy(fx * (by + 2)), nwin(sxy * (bz + 4)), nown(bx * by * bz) {}
  // whether the window of the brick at (i0, j0, k0) reaches beyond a line-tied face
  __device__ __forceinline__ bool at_face(const Geometry& g, int i0, int j0, int k0) const {
    return (g.bc[0] == BC_LINE_TIED && (i0 <= 1 || i0 + bx >= g.n[0] - 1)) ||
           (g.bc[1] == BC_LINE_TIED && (j0 <= 1 || j0 + by >= g.n[1] - 1)) ||
           (g.bc[2] == BC_LINE_TIED && (k0 <= 1 || k0 + bz >= g.n[2] - 1));
  }
};

struct BrickPoint {
  int index;  // grid index (0 off the grid)
  int ghost;  // step into the grid of a ghost point just beyond a line-tied face (0: none)
  int wraps;  // periodic wraps of x, y, z, each + 1, in bits 0-1, 2-3, 4-5; bit 6: on the grid
  __device__ __forceinline__ bool on() const { return wraps & 64; }
  __device__ __forceinline__ double wrap(int m) const { return (double)(((wraps >> (2 * m)) & 3) - 1); }
};

// window point e (past the window: off the grid, no ghost)
__device__ __forceinline__ BrickPoint brick_window(const Brick& b, const Geometry& g, int e, int i0, int j0, int k0) {
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int lz = small_div(e, b.sxy), e2 = e - lz * b.sxy, ly = small_div(e2, b.sx), lx = e2 - ly * b.sx;
  const int gi = i0 + lx - 2, gj = j0 + ly - 2, gk = k0 + lz - 2;
  const AxisIdx rx = resolve_near(gi, nx, g.bc[0]), ry = resolve_near(gj, ny, g.bc[1]);
  const AxisIdx rz = resolve_near(gk, nz, g.bc[2]);
  const bool in = e < b.nwin;
  BrickPoint p;
  const bool on = in && rx.ok && ry.ok && rz.ok;
  p.index = on ? (rz.i * ny + ry.i) * nx + rx.i : 0;
  p.wraps = (rx.w + 1) | (ry.w + 1) << 2 | (rz.w + 1) << 4 | (on ? 64 : 0);
  p.ghost = 0;
  if (in) {
    if (ry.ok && rz.ok && !rx.ok) p.ghost = gi == -1 ? 1 : (gi == nx ? -1 : 0);
    if (rx.ok && rz.ok && !ry.ok) p.ghost = gj == -1 ? b.sx : (gj == ny ? -b.sx : 0);
    if (rx.ok && ry.ok && !rz.ok) p.ghost = gk == -1 ? b.sxy : (gk == nz ? -b.sxy : 0);
  }
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
__device__ __forceinline__ BrickField brick_field(const Brick& b, const Geometry& g, int r, int tid, int i0, int j0,
                                                  int k0) {
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  int cx, cy, cz;  // field window coordinates
  bool in;
  if (r == 0) {
    in = tid < b.nown;
    const int e = in ? tid : 0;
    const int tz = small_div(e, b.bx * b.by), ty = small_div(e - tz * b.bx * b.by, b.bx);
    cx = e - (tz * b.by + ty) * b.bx + 1;
    cy = ty + 1;
    cz = tz + 1;
  } else {
    const int e = tid + (r - 1) * BRICK_THREADS, ring = 2 * (b.fx + b.by);
    if (e < 2 * b.fxy) {
      const int top = e >= b.fxy ? 1 : 0, e2 = e - top * b.fxy;
      cz = top * (b.bz + 1);
      cy = small_div(e2, b.fx);
      cx = e2 - cy * b.fx;
      in = true;
    } else {
      const int e2 = e - 2 * b.fxy, layer = small_div(e2, ring), e3 = e2 - layer * ring;
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
  const AxisIdx rx = resolve_near(i0 + cx - 1, nx, g.bc[0]), ry = resolve_near(j0 + cy - 1, ny, g.bc[1]);
  const AxisIdx rz = resolve_near(k0 + cz - 1, nz, g.bc[2]);
  BrickField p;
  const bool on = in && rx.ok && ry.ok && rz.ok;
  p.slot = in ? cz * b.fxy + cy * b.fx + cx : -1;
  p.window = (cz + 1) * b.sxy + (cy + 1) * b.sx + cx + 1;
  p.ends = on ? 64 : 0;
  if (r == 0 && in && i0 + cx - 1 < nx && j0 + cy - 1 < ny && k0 + cz - 1 < nz) p.ends |= 128;
  if (g.bc[0] == BC_LINE_TIED) p.ends |= rx.i == 0 ? 1 : (rx.i == nx - 1 ? 2 : 0);
  if (g.bc[1] == BC_LINE_TIED) p.ends |= ry.i == 0 ? 4 : (ry.i == ny - 1 ? 8 : 0);
  if (g.bc[2] == BC_LINE_TIED) p.ends |= rz.i == 0 ? 16 : (rz.i == nz - 1 ? 32 : 0);
  p.index = on ? (rz.i * ny + ry.i) * nx + rx.i : 0;
  return p;
}

}  // namespace relax
