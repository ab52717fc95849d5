// sweep_common.h -- device helpers shared by the forward stage sweeps (stage.hip) and the
// reverse sweeps (adjoint.hip): index resolution on line-tied and periodic axes, raw buffer
// accesses with masked-off lanes, the XCD-aware tile order, the 3x3 determinant, a
// Newton-refined reciprocal and reductions over a wave (also control.hip's).  Internal to the library.
#pragma once

#include "relax_device.h"

namespace relax {

// p mod 3 in [0, 3) for p >= -3072 (plane indices reach at most three planes below 0)
__device__ __forceinline__ int mod3(int p) { return (int)((unsigned)(p + 3072) % 3u); }

// e / d for 0 <= e < 2^21, 1 <= d: (e + 1/2) / d is at least 1 / (2 d) away from an integer, more than
// the 1.8e-7 (e + 1/2) / d that the reciprocal and the product round
__device__ __forceinline__ int small_div(int e, int d) {
  return (int)(((float)e + 0.5f) * __builtin_amdgcn_rcpf((float)d));
}

// One axis of a neighbour index: the in-range index, the number of periods wrapped (periodic
// axes), and whether the node exists (line-tied axes end at the boundary nodes).
struct AxisIdx {
  int i;
  int w;
  bool ok;
};

// Exact for v in [-n, 2n): the plane indices of a z march lie within three planes of [0, n) and
// n >= 4.  Other v give a wrong but in-range index on a periodic axis.
__device__ __forceinline__ AxisIdx resolve_near(int v, int n, int bc) {
  if (bc == BC_PERIODIC) {
    const int w = v < 0 ? -1 : (v >= n ? 1 : 0);
    return AxisIdx{min(max(v - w * n, 0), n - 1), w, true};
  }
  return AxisIdx{v, 0, v >= 0 && v < n};
}

// The same for a window's points, without a branch: at most one period away, others are off the grid.
// w is the wrap of a periodic axis, and 0 on a line-tied one.
__device__ __forceinline__ AxisIdx axis_index(int v, int n, int bc) {
  const int pn = bc == BC_PERIODIC ? n : 0, pw = bc == BC_PERIODIC ? 1 : 0;
  const int i = v + (v < 0 ? pn : (v >= n ? -pn : 0)), w = v < 0 ? -pw : (v >= n ? pw : 0);
  return AxisIdx{i, w, (unsigned)i < (unsigned)n};
}

// ---- buffer access --------------------------------------------------------------------------
// Element index of a masked-off lane: scaled by the element size it lands at or past the
// record count of every plane (a plane holds fewer than 2^28 nodes), so its load returns 0 and
// its store is dropped.
constexpr unsigned IE = 1u << 28;
constexpr int RSRC_WORD3 = 0x00020000;  // raw (untyped) buffer resource, gfx9 encoding
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// cache policy of the single-use accesses (node-wise loads and all stores): nt, non-temporal.
// The stencilled loads keep the default so that neighbouring tiles find their halo lines in L2.
constexpr int CPOL_STREAM = 2;

// resource for one component plane [base, base + nxy)
template <typename V>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const V* base, unsigned nxy) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<V*>(base), 0, (int)(nxy * sizeof(V)), RSRC_WORD3);
}
template <typename V, int CP = 0>
__device__ __forceinline__ V bload(__amdgpu_buffer_rsrc_t r, unsigned e) {
  if constexpr (sizeof(V) == 8)
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, (int)(e * 8u), 0, CP));
  else
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, (int)(e * 4u), 0, CP));
}
template <typename V>
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, unsigned e, V v) {
  if constexpr (sizeof(V) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)(e * 8u), 0, CPOL_STREAM);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)(e * 4u), 0, CPOL_STREAM);
}

// Gives v a register of its own here.  Without it a value carried over a load into the variable
// it came from may keep that variable's register: the load then goes elsewhere and is copied at
// the end of the loop, which waits for it at once.
template <typename V>
__device__ __forceinline__ void pin(V& v) {
  asm volatile("" : "+v"(v));
}

// v in other registers, which the result does not share even where v ends here: for a loaded value that a sum
// starts from.  The sum would be formed in its place, and the next load of it go elsewhere, as above.
__device__ __forceinline__ double taken(double v) {
  double r;
  asm volatile("v_mov_b64_e32 %0, %1" : "=&v"(r) : "v"(v));
  return r;
}

// logical tile of this workgroup; consecutive logical tiles share an XCD (the hardware
// hands workgroup b to XCD b mod 8), so neighbouring tiles reuse each other's halos in L2
__device__ __forceinline__ int logical_block(int bid, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int xcd = bid & 7, j = bid >> 3;
  return xcd * q + (xcd < r ? xcd : r) + j;
}

// The one-sided second-order row at a line-tied face, y0 the face node and y1, y2 the nodes inside it:
// (4 y1 - 3 y0) - y2 at the low end, y2 - (4 y1 - 3 y0) at the high end.  This is the sum in parentheses.  The
// row has one rounding, that of the sum, which lies inside the grid.  (A central difference with the ghost
// 3 (y0 - y1) + y2 would have that of the ghost, which lies outside: where a face is at a power of two, of
// half the accuracy.  51^3 on a box of +-4, +-4, +-10: u off by 4.4e-14 rms instead of 2.9e-14.)
__device__ __forceinline__ double face_sum(double y0, double y1) { return fma(-3.0, y0, 4.0 * y1); }

template <typename T>
__device__ __forceinline__ T det3(const T F[3][3]) {
  return F[0][0] * (F[1][1] * F[2][2] - F[1][2] * F[2][1]) - F[0][1] * (F[1][0] * F[2][2] - F[1][2] * F[2][0]) +
         F[0][2] * (F[1][0] * F[2][1] - F[1][1] * F[2][0]);
}

// 1/d by the hardware estimate and two Newton steps (d is a positive normal number here;
// d <= 0 means a folded cell, which the step control reports from det F itself)
__device__ __forceinline__ double rcp_nr(double d) {
  double r = __builtin_amdgcn_rcp(d);
  double e = fma(-d, r, 1.0);
  r = fma(r, e, r);
  e = fma(-d, r, 1.0);
  return fma(r, e, r);
}

__device__ __forceinline__ double max_nan(double a, double b) { return (b > a || b != b) ? b : a; }
__device__ __forceinline__ double min_nan(double a, double b) { return (b < a || b != b) ? b : a; }

// Reductions over a wave by DPP (four row shifts, then two row broadcasts): the result is in lane 63.
// idle: what a lane without a partner takes in.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double v, double idle) {
  typedef int i2 __attribute__((ext_vector_type(2)));
  const i2 a = __builtin_bit_cast(i2, v), z = __builtin_bit_cast(i2, idle);
  i2 r;
  r.x = __builtin_amdgcn_update_dpp(z.x, a.x, CTRL, ROWS, 0xf, false);
  r.y = __builtin_amdgcn_update_dpp(z.y, a.y, CTRL, ROWS, 0xf, false);
  return __builtin_bit_cast(double, r);
}
template <typename Op>
__device__ __forceinline__ double wave_reduce(double v, double idle, Op op) {
  v = op(v, dpp<0x111, 0xf>(v, idle));
  v = op(v, dpp<0x112, 0xf>(v, idle));
  v = op(v, dpp<0x114, 0xf>(v, idle));
  v = op(v, dpp<0x118, 0xf>(v, idle));
  v = op(v, dpp<0x142, 0xa>(v, idle));
  v = op(v, dpp<0x143, 0xc>(v, idle));
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
  return wave_reduce(v, 0.0, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_max(double v) { return wave_reduce(v, 0.0, max_nan); }  // v >= 0 or NaN
__device__ __forceinline__ double wave_min(double v) { return wave_reduce(v, INFINITY, min_nan); }

}  // namespace relax
