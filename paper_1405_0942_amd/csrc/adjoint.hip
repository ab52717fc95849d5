// adjoint.hip -- reverse-mode sweeps of the relaxation step (the transpose of stage.hip).
//
// Forward, per node n (unscaled differences, see stage.hip):
//   F'(n) = D y,  D' = det F',  rD = 1/D',  B = F' B0'' rD,
//   G'_a = B(n+e_a) - B(n-e_a),  c'_q = (F' e_b).G'_a - (F' e_a).G'_b,  w = c' rD,
//   J = F' w,  f = J x B,  u = gamma f (zero on line-tied faces).
// Reverse, given the cotangent ubar of u:
//   fbar = gamma ubar,  Jbar = B x fbar,  Bbar += fbar x J,
//   wbar = F'^T Jbar,   Fbar' += Jbar w^T,  cbar' = rD wbar,  rDbar += wbar . c',
//   Gbar'_x = cbar'_z F'_y - cbar'_y F'_z (and cyclic)  [F'_a = column a],
//   Fbar'_b += cbar'_q G'_a,  Fbar'_a -= cbar'_q G'_b,
//   Bbar(m) += sum_a Gbar'_a(m - e_a) - Gbar'_a(m + e_a)       (transpose of G'),
//   pull-back: Fbar' += (rD Bbar) B0''^T,  B0bar'' += F'^T Bbar rD,  rDbar += Bbar . F'B0'',
//   Dbar' = -rD^2 rDbar,  Fbar' += Dbar' cof(F'),
//   ybar = D^T Fbar'                                           (transpose of the differences).
// Gbar'(n) needs only F', rD, B and ubar at n, so Bbar(m) needs the stage input on a 2-node
// halo of m, the same footprint as the forward sweep.  adj_field_kernel forms Fbar' (9 values
// per node) and accumulates B0bar''; adj_gather_kernel applies D^T and, pointwise, assembles
// the cotangent of the previous stage's k (the Runge-Kutta transpose, see below).
//
// Runge-Kutta transpose of one step x_{n+1} = x_n + dt sum_s b5_s k_s, k_s = u(y_s),
// y_s = x_n + dt sum_{j<s} a_sj k_j:
//   kbar_s = dt (b5_s xbar_{n+1} + sum_{t>s} a_ts ybar_t),  ybar_s = (du/dy)(y_s)^T kbar_s,
//   xbar_n = xbar_{n+1} + sum_s ybar_s.
// The stage-6 field sweep scales xbar_{n+1} itself; the gather of stage t writes ybar_t and
// kbar_{t-1}, which the field sweep of stage t - 1 reads.
//
// Seeds (seed mode of adj_field_kernel): E_M = 1/2 sum zeta |B|^2 det F dV adds kappa D' B to
// Bbar and 1/2 kappa |B|^2 to Dbar' (kappa = zeta dV / (8 hx hy hz)); R2 = 1/2 sum_interior
// det F |f|^2 dV enters through ubar = det F dV f / gamma (read from a buffer) plus
// 1/2 |f|^2 dV / (8 hx hy hz) on Dbar'.
//
// The field sweep is laid out like the forward stage sweep: a 64 x 8 tile marching up a
// z-chunk, the stage input in an LDS ring of three planes (stages 3..6 stencil the stored
// y_s of the step), B in a ring of two planes, Gbar'_x and Gbar'_y in one plane that is
// transposed in-plane as soon as it is formed; buffer loads with masked-off lanes (offsets
// past the record count) issued one plane step ahead, so no divergent branch surrounds a
// memory instruction and the waits are exact.
#include "brick.h"

namespace relax {
namespace {

__device__ __forceinline__ void cross(const double a[3], const double b[3], double o[3]) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}

// B and the cotangents Gbar'_a = cotangent of G'_a (a = x, y, z) at a node from F', 1 / det F', B0'' and
// the cotangent ub of u (0 on line-tied faces)
__device__ __forceinline__ void transpose_field(const double F[3][3], double rD, const double b0[3], const double ub[3],
                                                double gamma, double B[3], double Gx[3], double Gy[3], double Gz[3]) {
#pragma unroll
  for (int m = 0; m < 3; m++) B[m] = (F[m][0] * b0[0] + F[m][1] * b0[1] + F[m][2] * b0[2]) * rD;
  const double fb[3] = {gamma * ub[0], gamma * ub[1], gamma * ub[2]};
  double Jb[3];
  cross(B, fb, Jb);
  double cb[3];  // cbar' = rD F'^T Jbar
#pragma unroll
  for (int n = 0; n < 3; n++) cb[n] = rD * (F[0][n] * Jb[0] + F[1][n] * Jb[1] + F[2][n] * Jb[2]);
#pragma unroll
  for (int m = 0; m < 3; m++) {
    Gx[m] = cb[2] * F[m][1] - cb[1] * F[m][2];
    Gy[m] = cb[0] * F[m][2] - cb[2] * F[m][0];
    Gz[m] = cb[1] * F[m][0] - cb[0] * F[m][1];
  }
}

// The transpose at one node: Fbar' (row-major) and the cotangent of B0'', from F', rD = 1 / det F', B,
// the cotangent ub of u, B0'', the differences G[a][m] of B (0 on line-tied faces, where J = 0), and
// Bt = the transpose of G'.  zeta: the energy weight of the node (SEED).
template <bool SEED>
__device__ __forceinline__ void transpose_node(const double F[3][3], double rD, const double B[3], const double ub[3],
                                               const double b0[3], const double G[3][3], const double Bt[3],
                                               bool interior, double zeta, const AdjArgs& a, double Fbar[9],
                                               double dB0[3]) {
  double Bb[3] = {0, 0, 0};
  double Fb[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  double rDb = 0.0, Db_direct = 0.0;
  if (interior) {
    double cq[3];
    cq[0] = F[0][2] * G[1][0] + F[1][2] * G[1][1] + F[2][2] * G[1][2] -
            (F[0][1] * G[2][0] + F[1][1] * G[2][1] + F[2][1] * G[2][2]);
    cq[1] = F[0][0] * G[2][0] + F[1][0] * G[2][1] + F[2][0] * G[2][2] -
            (F[0][2] * G[0][0] + F[1][2] * G[0][1] + F[2][2] * G[0][2]);
    cq[2] = F[0][1] * G[0][0] + F[1][1] * G[0][1] + F[2][1] * G[0][2] -
            (F[0][0] * G[1][0] + F[1][0] * G[1][1] + F[2][0] * G[1][2]);
    const double w[3] = {cq[0] * rD, cq[1] * rD, cq[2] * rD};
    double J[3];
#pragma unroll
    for (int m = 0; m < 3; m++) J[m] = F[m][0] * w[0] + F[m][1] * w[1] + F[m][2] * w[2];
    const double fb[3] = {a.gamma * ub[0], a.gamma * ub[1], a.gamma * ub[2]};
    double Jb[3], t3[3];
    cross(B, fb, Jb);
    cross(fb, J, t3);
#pragma unroll
    for (int m = 0; m < 3; m++) Bb[m] += t3[m];
    double wb[3];
#pragma unroll
    for (int n = 0; n < 3; n++) wb[n] = F[0][n] * Jb[0] + F[1][n] * Jb[1] + F[2][n] * Jb[2];
#pragma unroll
    for (int m = 0; m < 3; m++)
#pragma unroll
      for (int n = 0; n < 3; n++) Fb[m][n] += Jb[m] * w[n];
    const double cb[3] = {wb[0] * rD, wb[1] * rD, wb[2] * rD};
    rDb += wb[0] * cq[0] + wb[1] * cq[1] + wb[2] * cq[2];
    // c'_q = F'_b . G'_a - F'_a . G'_b for (a, b, q) = (1, 2, 0), (2, 0, 1), (0, 1, 2)
#pragma unroll
    for (int m = 0; m < 3; m++) {
      Fb[m][2] += cb[0] * G[1][m];
      Fb[m][1] -= cb[0] * G[2][m];
      Fb[m][0] += cb[1] * G[2][m];
      Fb[m][2] -= cb[1] * G[0][m];
      Fb[m][1] += cb[2] * G[0][m];
      Fb[m][0] -= cb[2] * G[1][m];
    }
    if constexpr (SEED) {
      double f[3];
      cross(J, B, f);
      Db_direct += a.seed_R2 * 0.5 * a.g.dV * a.g.inv8h3 * (f[0] * f[0] + f[1] * f[1] + f[2] * f[2]);
    }
  }
#pragma unroll
  for (int m = 0; m < 3; m++) Bb[m] += Bt[m];
  if constexpr (SEED) {
    const double kappa = a.seed_EM * zeta * a.g.dV * a.g.inv8h3;
    const double D = 1.0 / rD;
#pragma unroll
    for (int m = 0; m < 3; m++) Bb[m] += kappa * D * B[m];
    Db_direct += 0.5 * kappa * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2]);
  }
  // pull-back B = F' B0'' rD
  double v[3];
#pragma unroll
  for (int m = 0; m < 3; m++) v[m] = F[m][0] * b0[0] + F[m][1] * b0[1] + F[m][2] * b0[2];
  rDb += Bb[0] * v[0] + Bb[1] * v[1] + Bb[2] * v[2];
#pragma unroll
  for (int m = 0; m < 3; m++)
#pragma unroll
    for (int n = 0; n < 3; n++) Fb[m][n] += rD * Bb[m] * b0[n];
#pragma unroll
  for (int n = 0; n < 3; n++) dB0[n] = rD * (F[0][n] * Bb[0] + F[1][n] * Bb[1] + F[2][n] * Bb[2]);
  // det: Dbar' cof(F')
  const double Db = -rD * rD * rDb + Db_direct;
#pragma unroll
  for (int m = 0; m < 3; m++)
#pragma unroll
    for (int n = 0; n < 3; n++) {
      const int m1 = (m + 1) % 3, m2 = (m + 2) % 3, n1 = (n + 1) % 3, n2 = (n + 2) % 3;
      Fbar[3 * m + n] = Fb[m][n] + Db * (F[m1][n1] * F[m2][n2] - F[m1][n2] * F[m2][n1]);
    }
}

template <int S, bool XYP, bool SEED>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void adj_field_kernel(AdjArgs a) {
  constexpr bool WK = (!SEED && S == 2);  // the window carries k_1 too
  constexpr int NP2 = (RY2 * RX2 + NTHREADS - 1) / NTHREADS;
  constexpr int NP1 = (RY1 * RX1 + NTHREADS - 1) / NTHREADS;

  const Geometry& g = a.g;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const long long N = g.N;
  const unsigned nxy = (unsigned)nx * (unsigned)ny;
  const int bcx = XYP ? BC_PERIODIC : g.bc[0];
  const int bcy = XYP ? BC_PERIODIC : g.bc[1];
  const int bcz = g.bc[2];
  const double gamma = a.gamma;

  const double dt = SEED ? 0.0 : *a.dt;
  const double c21 = dt * CK::a[1][0];
  // the cotangent of u: seed buffer, dt b5_6 xbar_{n+1} (stage 6), or the gathered kbar_s
  const bool v_on = !SEED || a.useed != nullptr;
  const double* __restrict__ vsrc = SEED ? (a.useed ? a.useed : a.B0) : (S == 6 ? a.xbar : a.ubar);
  const double cv = (!SEED && S == 6) ? dt * CK::b5[5] : 1.0;
  const double* __restrict__ wsrc = (SEED || S <= 2) ? a.x : a.y[S > 2 ? S - 3 : 0];
  const double* __restrict__ k1p = a.k[0];

  const int lb = logical_block(blockIdx.x, g.nblocks);
  const int tile_x = lb % g.tiles[0];
  const int tile_y = (lb / g.tiles[0]) % g.tiles[1];
  const int chunk = lb / (g.tiles[0] * g.tiles[1]);
  const int i0 = tile_x * TX, j0 = tile_y * TY;
  const int z0 = chunk * g.tz;
  const int z1 = min(z0 + g.tz, nz);
  const int tid = threadIdx.x;
  const int tx = tid % TX, ty = tid / TX;

  __shared__ double ys[3][3][RY2 * RX2];  // stage input, ring of 3 planes
  __shared__ double bs[2][3][RY1 * RX1];  // B, ring of 2 planes
  __shared__ double gxy[6][RY1 * RX1];    // Gbar'_x (0..2) and Gbar'_y (3..5) of the newest plane

  auto zload = [&](int pz) {
    if (bcz == BC_PERIODIC) return resolve_near(pz, nz, bcz).i;
    return min(max(pz, 0), nz - 1);
  };

  // index tables (as in the forward sweep)
  unsigned w2e[NP2];
  int w2w[NP2];
#pragma unroll
  for (int r = 0; r < NP2; r++) {
    const int e = tid + r * NTHREADS;
    const int row = e / RX2, col = e - row * RX2;
    const AxisIdx rx = resolve(i0 + col - 2, nx, bcx), ry = resolve(j0 + row - 2, ny, bcy);
    w2e[r] = (e < RY2 * RX2 && rx.ok && ry.ok) ? (unsigned)(ry.i * nx + rx.i) : IE;
    w2w[r] = (ry.w << 16) + (rx.w & 0xffff);
  }
  unsigned f1e[NP1];
  int f1r[NP1], f1c[NP1];
#pragma unroll
  for (int r = 0; r < NP1; r++) {
    const int e = tid + r * NTHREADS;
    int r1, c1;
    if (e < NTHREADS) {
      r1 = e / TX + 1;
      c1 = e % TX + 1;
    } else {
      const int e2 = e - NTHREADS;
      if (e2 < RX1) {
        r1 = 0;
        c1 = e2;
      } else if (e2 < 2 * RX1) {
        r1 = RY1 - 1;
        c1 = e2 - RX1;
      } else {
        const int e3 = e2 - 2 * RX1;
        r1 = 1 + (e3 >> 1);
        c1 = (e3 & 1) ? RX1 - 1 : 0;
      }
    }
    const AxisIdx rx = resolve(i0 + c1 - 1, nx, bcx), ry = resolve(j0 + r1 - 1, ny, bcy);
    f1e[r] = (e < RY1 * RX1 && rx.ok && ry.ok) ? (unsigned)(ry.i * nx + rx.i) : IE;
    f1r[r] = (e < RY1 * RX1) ? r1 : -1;
    f1c[r] = c1;
  }
  const int gi_t = i0 + tx, gj_t = j0 + ty;
  const bool tile_ok = (gi_t < nx) && (gj_t < ny);
  const unsigned out_e = tile_ok ? (unsigned)(gj_t * nx + gi_t) : IE;

  auto face_at = [&](int gi, int gj, int p) {
    return (bcx == BC_LINE_TIED && (gi == 0 || gi == nx - 1)) || (bcy == BC_LINE_TIED && (gj == 0 || gj == ny - 1)) ||
           (bcz == BC_LINE_TIED && (p == 0 || p == nz - 1));
  };

  // ---- loads, issued one plane step ahead of their use ---------------------------------------
  double wx[NP2][3];
  double wk[WK ? NP2 : 1][3];
  double b0r[NP1][3], vr[NP1][3];
  double bbr[3];  // B0bar'' at the output node
  auto load_window = [&](int pz) {
    const long long zo = (long long)zload(pz) * nxy;
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const auto rs = plane_rsrc(wsrc + m * N + zo, nxy);
#pragma unroll
      for (int r = 0; r < NP2; r++) wx[r][m] = bload<double>(rs, w2e[r]);
    }
    if constexpr (WK) {
#pragma unroll
      for (int m = 0; m < 3; m++) {
        const auto rs = plane_rsrc(k1p + m * N + zo, nxy);
#pragma unroll
        for (int r = 0; r < NP2; r++) wk[r][m] = bload<double>(rs, w2e[r]);
      }
    }
  };
  auto commit_window = [&](int pz) {
    const AxisIdx rz = resolve_near(pz, nz, bcz);
    const int slot = mod3(pz);
    const double shz = rz.w * g.period[2];
#pragma unroll
    for (int r = 0; r < NP2; r++) {
      const int e = tid + r * NTHREADS;
      const bool ok = (w2e[r] != IE);
      double v[3];
#pragma unroll
      for (int m = 0; m < 3; m++) {
        double y = wx[r][m];
        if constexpr (WK) y = fma(c21, wk[r][m], y);
        v[m] = y;
      }
      v[0] += (double)(short)(w2w[r] & 0xffff) * g.period[0];
      v[1] += (double)(w2w[r] >> 16) * g.period[1];
      v[2] += shz;
      if (e < RY2 * RX2) {
#pragma unroll
        for (int m = 0; m < 3; m++) ys[slot][m][e] = ok ? v[m] : 0.0;
      }
    }
  };
  auto load_field = [&](int pz) {
    const long long zo = (long long)zload(pz) * nxy;
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const auto rb = plane_rsrc(a.B0 + m * N + zo, nxy);
      const auto rv = plane_rsrc(vsrc + m * N + zo, nxy);
#pragma unroll
      for (int r = 0; r < NP1; r++) {
        b0r[r][m] = bload<double>(rb, f1e[r]);
        vr[r][m] = bload<double>(rv, v_on ? f1e[r] : IE);
      }
    }
  };
  auto load_point = [&](int pz) {
    const bool on = (pz >= z0 && pz < z1);
    const long long zo = (long long)zload(pz) * nxy;
#pragma unroll
    for (int m = 0; m < 3; m++) bbr[m] = bload<double, CPOL_STREAM>(plane_rsrc(a.B0bar + m * N + zo, nxy), on ? out_e : IE);
  };
  double so_F[9], so_B[3];
#pragma unroll
  for (int i = 0; i < 9; i++) so_F[i] = 0.0;
#pragma unroll
  for (int m = 0; m < 3; m++) so_B[m] = 0.0;
  auto store_point = [&](int qz, bool on) {
    const long long zo = (long long)zload(qz) * nxy;
    const unsigned eo = on ? out_e : IE;
#pragma unroll
    for (int i = 0; i < 9; i++) bstore(plane_rsrc(a.Fbar + i * N + zo, nxy), eo, so_F[i]);
#pragma unroll
    for (int m = 0; m < 3; m++) bstore(plane_rsrc(a.B0bar + m * N + zo, nxy), eo, so_B[m]);
  };

  auto jac_xy = [&](int r, int c, int p, int gi, int gj, double F[3][3]) {
    const int o = r * RX2 + c;
    const int sp = mod3(p);
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const double* yc = ys[sp][m];
      if (XYP || bcx == BC_PERIODIC || (gi > 0 && gi < nx - 1))
        F[m][0] = yc[o + 1] - yc[o - 1];
      else if (gi == 0)
        F[m][0] = -3.0 * yc[o] + 4.0 * yc[o + 1] - yc[o + 2];
      else
        F[m][0] = 3.0 * yc[o] - 4.0 * yc[o - 1] + yc[o - 2];
      if (XYP || bcy == BC_PERIODIC || (gj > 0 && gj < ny - 1))
        F[m][1] = yc[o + RX2] - yc[o - RX2];
      else if (gj == 0)
        F[m][1] = -3.0 * yc[o] + 4.0 * yc[o + RX2] - yc[o + 2 * RX2];
      else
        F[m][1] = 3.0 * yc[o] - 4.0 * yc[o - RX2] + yc[o - 2 * RX2];
    }
  };
  auto jacobian = [&](int r, int c, int p, int gi, int gj, double F[3][3]) {
    jac_xy(r, c, p, gi, gj, F);
    const int o = r * RX2 + c;
    if (bcz == BC_PERIODIC || (p > 0 && p < nz - 1)) {
      const int sa = mod3(p + 1), sb = mod3(p - 1);
#pragma unroll
      for (int m = 0; m < 3; m++) F[m][2] = ys[sa][m][o] - ys[sb][m][o];
    } else if (p == 0) {
#pragma unroll
      for (int m = 0; m < 3; m++) F[m][2] = -3.0 * ys[0][m][o] + 4.0 * ys[1][m][o] - ys[2][m][o];
    } else {
      const int s0 = mod3(p), s1 = mod3(p - 1), s2 = mod3(p - 2);
#pragma unroll
      for (int m = 0; m < 3; m++) F[m][2] = 3.0 * ys[s0][m][o] - 4.0 * ys[s1][m][o] + ys[s2][m][o];
    }
  };

  const bool perz = (bcz == BC_PERIODIC);
  const int pb0 = perz ? z0 - 1 : max(z0 - 1, 0);
  const int pb1 = perz ? z1 : min(z1, nz - 1);
  auto need_hi = [&](int p) { return perz ? p + 1 : (p == 0 ? 2 : (p == nz - 1 ? p : p + 1)); };
  auto need_lo = [&](int p) { return perz ? p - 1 : (p == 0 ? 0 : (p == nz - 1 ? p - 2 : p - 1)); };

  // prologue: the first stage-input window, then the loads and (dropped) stores a plane step
  // leaves in flight, in the same order
  int hi = need_hi(pb0);
  for (int pz = need_lo(pb0); pz <= hi; pz++) {
    load_window(pz);
    commit_window(pz);
  }
  __syncthreads();
  load_field(pb0);
  load_window(hi + 1);
  load_point(pb0 - 1);
  store_point(pb0 - 1, false);

  // own-node values carried between plane steps (q = p - 1 is the output plane)
  double Fzq[3] = {0, 0, 0};  // z column of F' at q (the x and y columns are re-read from the ring)
  double rDq = 0.0;
  double ubq[3] = {0, 0, 0}, Bq[3] = {0, 0, 0}, Bqm[3] = {0, 0, 0}, b0q[3] = {0, 0, 0};
  double gzqm[3] = {0, 0, 0}, gzq[3] = {0, 0, 0};  // Gbar'_z at q - 1 and q
  double Bbxyq[3] = {0, 0, 0};                     // in-plane transpose of Gbar' at q
  const int ot = (ty + 1) * RX1 + (tx + 1);

  for (int p = pb0; p <= z1; p++) {
    const int q = p - 1;
    const bool qout = (q >= z0 && q < z1);
    // 1. B, Gbar'_x, Gbar'_y on the tile + 1-node halo of plane p; own-node values
    double Fzp[3] = {0, 0, 0};
    double rDp = 0.0, ubp[3] = {0, 0, 0}, Bp[3] = {0, 0, 0}, b0p[3] = {0, 0, 0}, gzp[3] = {0, 0, 0};
    if (p <= pb1) {
      const int sb = p & 1;
#pragma unroll
      for (int r = 0; r < NP1; r++) {
        __builtin_amdgcn_sched_barrier(0);
        if (f1r[r] >= 0) {
          const int r1 = f1r[r], c1 = f1c[r];
          const int gi = i0 + c1 - 1, gj = j0 + r1 - 1;
          double B[3] = {0, 0, 0}, Gx[3] = {0, 0, 0}, Gy[3] = {0, 0, 0}, Gz[3] = {0, 0, 0}, ub[3] = {0, 0, 0};
          if (f1e[r] != IE) {
            double F[3][3];
            jacobian(r1 + 1, c1 + 1, p, gi, gj, F);
            const double rD = rcp_nr(det3(F));
            const bool live = !face_at(gi, gj, p);
#pragma unroll
            for (int m = 0; m < 3; m++) ub[m] = live ? cv * vr[r][m] : 0.0;
            transpose_field(F, rD, b0r[r], ub, gamma, B, Gx, Gy, Gz);
            if (r == 0) {
#pragma unroll
              for (int m = 0; m < 3; m++) {
                Fzp[m] = F[m][2];
                ubp[m] = ub[m];
                Bp[m] = B[m];
                b0p[m] = b0r[r][m];
                gzp[m] = Gz[m];
              }
              rDp = rD;
            }
          }
          const int o = r1 * RX1 + c1;
#pragma unroll
          for (int m = 0; m < 3; m++) {
            bs[sb][m][o] = B[m];
            gxy[m][o] = Gx[m];
            gxy[3 + m][o] = Gy[m];
          }
        }
      }
    }
    load_field(p + 1 <= pb1 ? p + 1 : pb1);
    // x and y columns of F' at the own node of plane q, read before the barrier: the commit
    // below reuses plane q's ring slot
    double F[3][3];
    if (qout) {
      jac_xy(ty + 2, tx + 2, q, gi_t, gj_t, F);
#pragma unroll
      for (int m = 0; m < 3; m++) F[m][2] = Fzq[m];
    }
    __syncthreads();

    // 2. commit the stage-input plane field(p + 1) needs; issue the next one
    if (p + 1 <= pb1 && need_hi(p + 1) > hi) {
      hi++;
      commit_window(hi);
    }
    load_window(hi + 1);

    // 3. in-plane transpose of Gbar' at the own node of plane p (used by the next step)
    double Bbxyp[3];
#pragma unroll
    for (int m = 0; m < 3; m++)
      Bbxyp[m] = (gxy[m][ot - 1] - gxy[m][ot + 1]) + (gxy[3 + m][ot - RX1] - gxy[3 + m][ot + RX1]);

    // 4. the transpose at the own node of plane q
    if (qout) {
      const bool interior = !face_at(gi_t, gj_t, q);
      double G[3][3] = {};  // G[a][m]
      if (interior) {
        const int sq = q & 1;
#pragma unroll
        for (int m = 0; m < 3; m++) {
          G[0][m] = bs[sq][m][ot + 1] - bs[sq][m][ot - 1];
          G[1][m] = bs[sq][m][ot + RX1] - bs[sq][m][ot - RX1];
          G[2][m] = Bp[m] - Bqm[m];
        }
      }
      double Bt[3];  // transpose of G': sum_a Gbar'_a(m - e_a) - Gbar'_a(m + e_a)
#pragma unroll
      for (int m = 0; m < 3; m++) Bt[m] = Bbxyq[m] + (gzqm[m] - gzp[m]);
      double zeta = 1.0;
      if constexpr (SEED) {
        if (bcx == BC_LINE_TIED && (gi_t == 0 || gi_t == nx - 1)) zeta *= 0.5;
        if (bcy == BC_LINE_TIED && (gj_t == 0 || gj_t == ny - 1)) zeta *= 0.5;
        if (bcz == BC_LINE_TIED && (q == 0 || q == nz - 1)) zeta *= 0.5;
      }
      double dB[3];
      transpose_node<SEED>(F, rDq, Bq, ubq, b0q, G, Bt, interior, zeta, a, so_F, dB);
#pragma unroll
      for (int m = 0; m < 3; m++) so_B[m] = bbr[m] + dB[m];
    }
    load_point(p);  // B0bar'' at the output node of the next plane step
    store_point(q, qout);
    __syncthreads();

#pragma unroll
    for (int m = 0; m < 3; m++) {
      Fzq[m] = Fzp[m];
      ubq[m] = ubp[m];
      Bqm[m] = Bq[m];
      Bq[m] = Bp[m];
      b0q[m] = b0p[m];
      gzqm[m] = gzq[m];
      gzq[m] = gzp[m];
      Bbxyq[m] = Bbxyp[m];
    }
    rDq = rDp;
  }
}

// The same for small grids, a brick of nodes per workgroup (see brick.hip): the stage input with its
// 2-node halo, B and the three Gbar' on the brick and its 1-node halo, all planes at once, two or three
// barriers.  LDS: up to 157 KB (Gbar' takes 72 bytes a field point), one workgroup per CU.  Up to
// 600 000 nodes (make_adj_geometry): us per step of a backward pass, march / bricks: 16^3 714 / 145,
// 33^3 846 / 173, 64^3 606 / 322, 81^3 line-tied 1034 / 703, 64 x 64 x 192 731 / 797, 128^3 1580 / 2187.
constexpr int NPW = (ADJ_WINDOW + BRICK_THREADS - 1) / BRICK_THREADS;
constexpr int NPF = 1 + (BRICK_SHELL + BRICK_THREADS - 1) / BRICK_THREADS;

template <int S, bool SEED>
__global__ __launch_bounds__(BRICK_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void adj_brick_kernel(AdjArgs a) {
  constexpr bool WK = (!SEED && S == 2);
  const Geometry& g = a.g;
  const long long N = g.N;
  const Brick br(g);
  const int lb = logical_block(blockIdx.x, g.nblocks);
  const int i0 = (lb % g.tiles[0]) * br.bx;
  const int j0 = ((lb / g.tiles[0]) % g.tiles[1]) * br.by;
  const int k0 = (lb / (g.tiles[0] * g.tiles[1])) * br.bz;
  const int tid = threadIdx.x;
  const double dt = SEED ? 0.0 : *a.dt;
  const double c21 = dt * CK::a[1][0];
  const bool v_on = !SEED || a.useed != nullptr;
  const double* __restrict__ vsrc = SEED ? (a.useed ? a.useed : a.B0) : (S == 6 ? a.xbar : a.ubar);
  const double cv = v_on ? ((!SEED && S == 6) ? dt * CK::b5[5] : 1.0) : 0.0;
  const double* __restrict__ wsrc = (SEED || S <= 2) ? a.x : a.y[S > 2 ? S - 3 : 0];

  __shared__ double ys[3][ADJ_WINDOW];
  __shared__ double bs[3][BRICK_FIELD];
  __shared__ double gs[9][BRICK_FIELD];

  // ---- all loads first
  double wx[NPW][3], wk[WK ? NPW : 1][3];
  BrickPoint wp[NPW];
#pragma unroll
  for (int r = 0; r < NPW; r++) {
    wp[r] = brick_window(br, g, tid + r * BRICK_THREADS, i0, j0, k0);
    const int i = wp[r].index;
#pragma unroll
    for (int m = 0; m < 3; m++) wx[r][m] = wsrc[m * N + i];
    if constexpr (WK) {
#pragma unroll
      for (int m = 0; m < 3; m++) wk[r][m] = a.k[0][m * N + i];
    }
  }
  double b0r[NPF][3], vr[NPF][3];
  BrickField fp[NPF];
#pragma unroll
  for (int r = 0; r < NPF; r++) {
    fp[r] = brick_field(br, g, r, tid, i0, j0, k0);
#pragma unroll
    for (int m = 0; m < 3; m++) {
      b0r[r][m] = a.B0[m * N + fp[r].index];
      vr[r][m] = vsrc[m * N + fp[r].index];
    }
  }
  const bool node = fp[0].node();
  const int own = fp[0].index;
  double bbr[3];
#pragma unroll
  for (int m = 0; m < 3; m++) bbr[m] = a.B0bar[m * N + own];

  // ---- stage input
#pragma unroll
  for (int r = 0; r < NPW; r++) {
    const int e = tid + r * BRICK_THREADS;
    if (e < br.nwin) {
#pragma unroll
      for (int m = 0; m < 3; m++) {
        double y = wx[r][m];
        if constexpr (WK) y = fma(c21, wk[r][m], y);
        ys[m][e] = wp[r].on() ? y + wp[r].wrap(m) * g.period[m] : 0.0;
      }
    }
  }
  __syncthreads();
  if (br.at_face(g, i0, j0, k0)) {
#pragma unroll
    for (int r = 0; r < NPW; r++) {
      const int e = tid + r * BRICK_THREADS, s = wp[r].ghost;
      if (s != 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) ys[m][e] = fma(3.0, ys[m][e + s] - ys[m][e + 2 * s], ys[m][e + 3 * s]);
      }
    }
    __syncthreads();
  }

  // ---- B and Gbar' on the brick and its 1-node halo
  double Fq[3][3], Bq[3], ubq[3], rDq;
#pragma unroll
  for (int r = 0; r < NPF; r++) {
    if (r == 0 || fp[r].slot >= 0) {
      const int o = fp[r].window;
      double F[3][3], B[3], Gx[3], Gy[3], Gz[3], ub[3];
#pragma unroll
      for (int m = 0; m < 3; m++) {
        F[m][0] = ys[m][o + 1] - ys[m][o - 1];
        F[m][1] = ys[m][o + br.sx] - ys[m][o - br.sx];
        F[m][2] = ys[m][o + br.sxy] - ys[m][o - br.sxy];
      }
      const double rD = fp[r].on() ? rcp_nr(det3(F)) : 0.0;
      const bool live = fp[r].on() && !fp[r].face();
#pragma unroll
      for (int m = 0; m < 3; m++) ub[m] = live ? cv * vr[r][m] : 0.0;
      transpose_field(F, rD, b0r[r], ub, a.gamma, B, Gx, Gy, Gz);
      if (r == 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) {
#pragma unroll
          for (int c = 0; c < 3; c++) Fq[m][c] = F[m][c];
          Bq[m] = B[m];
          ubq[m] = ub[m];
        }
        rDq = rD;
      }
      if (fp[r].slot >= 0) {
        const int f = fp[r].slot;
#pragma unroll
        for (int m = 0; m < 3; m++) {
          bs[m][f] = B[m];
          gs[m][f] = Gx[m];
          gs[3 + m][f] = Gy[m];
          gs[6 + m][f] = Gz[m];
        }
      }
    }
  }
  __syncthreads();
  if (!node) return;

  // ---- the transpose at the own node
  const int o = fp[0].slot, fx = br.fx, fxy = br.fxy;
  const bool interior = !fp[0].face();
  double G[3][3] = {}, Bt[3];
#pragma unroll
  for (int m = 0; m < 3; m++) {
    if (interior) {
      G[0][m] = bs[m][o + 1] - bs[m][o - 1];
      G[1][m] = bs[m][o + fx] - bs[m][o - fx];
      G[2][m] = bs[m][o + fxy] - bs[m][o - fxy];
    }
    Bt[m] = (gs[m][o - 1] - gs[m][o + 1]) + (gs[3 + m][o - fx] - gs[3 + m][o + fx]) +
            (gs[6 + m][o - fxy] - gs[6 + m][o + fxy]);
  }
  double zeta = 1.0;
  if constexpr (SEED) zeta = (fp[0].ends & 3 ? 0.5 : 1.0) * (fp[0].ends & 12 ? 0.5 : 1.0) * (fp[0].ends & 48 ? 0.5 : 1.0);
  double Fb[9], dB[3];
  transpose_node<SEED>(Fq, rDq, Bq, ubq, b0r[0], G, Bt, interior, zeta, a, Fb, dB);
#pragma unroll
  for (int i = 0; i < 9; i++) a.Fbar[i * N + own] = Fb[i];
#pragma unroll
  for (int m = 0; m < 3; m++) a.B0bar[m * N + own] = bbr[m] + dB[m];
}

// ybar = D^T Fbar': each column a of Fbar' is pulled back along axis a with the transposed
// difference rows (central: +1 at n+e_a, -1 at n-e_a; one-sided ends: (-3, 4, -1) and (3, -4, 1)).
// MODE 0 (stage STAGE >= 2): ybar_t = D^T Fbar' -> ybar_out, and the cotangent of k_{t-1},
//   dt (b5_{t-1} xbar + sum_{t' >= t} a_{t',t-1} ybar_{t'}) -> ubar_out;
// MODE 1 (stage 1): xbar += D^T Fbar' + sum_{t=2..6} ybar_t;  MODE 2 (seed): xbar = D^T Fbar'.
// Bound by its 190 to 290 bytes a node: one thread a node, rows of 64 along x so that every access is
// coalesced and no index needs a 64-bit division (64 x 64 x 192: 29 us; 16^3: 8 -> 4 us against a
// grid-stride loop with 64-bit divisions).
template <int MODE, int STAGE>
__global__ __launch_bounds__(256) void adj_gather_kernel(AdjArgs a, int bxs, int bys) {
  const Geometry& g = a.g;
  const long long N = g.N;
  const int nx = g.n[0], ny = g.n[1];
  const int lb = logical_block(blockIdx.x, gridDim.x);
  const int k = lb / (bxs * bys), rem = lb - k * bxs * bys, jb = rem / bxs;
  const int i = (rem - jb * bxs) * 64 + (threadIdx.x & 63), j = jb * 4 + (threadIdx.x >> 6);
  if (i >= nx || j >= ny) return;
  const long long p = ((long long)k * ny + j) * nx + i;
  const double dt = (MODE == 0) ? *a.dt : 0.0;
  double yb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int ax = 0; ax < 3; ax++) {
    const int n = g.n[ax], v = ax == 0 ? i : (ax == 1 ? j : k);
    const long long stride = ax == 0 ? 1 : (ax == 1 ? (long long)nx : (long long)nx * ny);
    auto col = [&](int vv, double c) {  // yb += c * Fbar'[:, ax] at the node with index vv along ax
      const long long m = p + (long long)(vv - v) * stride;
#pragma unroll
      for (int r = 0; r < 3; r++) yb[r] += c * a.Fbar[(3 * r + ax) * N + m];
    };
    if (g.bc[ax] == BC_PERIODIC) {
      col(v == 0 ? n - 1 : v - 1, 1.0);
      col(v == n - 1 ? 0 : v + 1, -1.0);
    } else {
      if (v - 1 >= 1 && v - 1 <= n - 2) col(v - 1, 1.0);
      if (v + 1 >= 1 && v + 1 <= n - 2) col(v + 1, -1.0);
      if (v == 0) col(0, -3.0);
      if (v == 1) col(0, 4.0);
      if (v == 2) col(0, -1.0);
      if (v == n - 1) col(n - 1, 3.0);
      if (v == n - 2) col(n - 1, -4.0);
      if (v == n - 3) col(n - 1, 1.0);
    }
  }
#pragma unroll
  for (int r = 0; r < 3; r++) {
    if constexpr (MODE == 0) {
      constexpr int s = STAGE - 1;  // the stage whose k's cotangent is assembled
      a.ybar_out[p + r * N] = yb[r];
      double v = CK::b5[s - 1] * a.xbar[p + r * N] + CK::a[STAGE - 1][s - 1] * yb[r];
#pragma unroll
      for (int t = STAGE + 1; t <= 6; t++) v += CK::a[t - 1][s - 1] * a.ybar[t][p + r * N];
      a.ubar_out[p + r * N] = dt * v;
    } else if constexpr (MODE == 1) {
      double s = a.xbar_out[p + r * N] + yb[r];
#pragma unroll
      for (int t = 2; t <= 6; t++) s += a.ybar[t][p + r * N];
      a.xbar_out[p + r * N] = s;
    } else {
      a.xbar_out[p + r * N] = yb[r];
    }
  }
}

__global__ void fill_kernel(double* __restrict__ v, long long n, double val) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    v[i] = val;
}

// the forward recompute of one recorded step runs on its own control block
__global__ void seg_step_kernel(Control* c2, const double* __restrict__ dt_record, long long n) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    c2->dt = dt_record[n];
    c2->status = 0;
    c2->cur = 0;
    c2->accepted = 0;
    c2->target = 1;
    c2->need_k1 = 1;
    c2->record = 0;
  }
}

template <int S, bool XYP, bool SEED>
hipError_t launch_field_t(const AdjArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((adj_field_kernel<S, XYP, SEED>), dim3(a.g.nblocks), dim3(NTHREADS), 0, st, a);
  return hipGetLastError();
}

template <bool XYP>
hipError_t launch_field_x(int s, bool seed, const AdjArgs& a, hipStream_t st) {
  if (seed) return launch_field_t<1, XYP, true>(a, st);
  switch (s) {
    case 1: return launch_field_t<1, XYP, false>(a, st);
    case 2: return launch_field_t<2, XYP, false>(a, st);
    case 3: return launch_field_t<3, XYP, false>(a, st);
    case 4: return launch_field_t<4, XYP, false>(a, st);
    case 5: return launch_field_t<5, XYP, false>(a, st);
    case 6: return launch_field_t<6, XYP, false>(a, st);
    default: return hipErrorInvalidValue;
  }
}

unsigned grid_for(long long n) {
  long long b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (unsigned)b;
}

}  // namespace

hipError_t launch_adj_field(int s, bool seed, const AdjArgs& a, hipStream_t st) {
  if (a.g.brick[0]) {
    const dim3 grid(a.g.nblocks), block(BRICK_THREADS);
    switch (seed ? 0 : s) {
      case 0: hipLaunchKernelGGL((adj_brick_kernel<1, true>), grid, block, 0, st, a); break;
      case 1: hipLaunchKernelGGL((adj_brick_kernel<1, false>), grid, block, 0, st, a); break;
      case 2: hipLaunchKernelGGL((adj_brick_kernel<2, false>), grid, block, 0, st, a); break;
      case 3: hipLaunchKernelGGL((adj_brick_kernel<3, false>), grid, block, 0, st, a); break;
      case 4: hipLaunchKernelGGL((adj_brick_kernel<4, false>), grid, block, 0, st, a); break;
      case 5: hipLaunchKernelGGL((adj_brick_kernel<5, false>), grid, block, 0, st, a); break;
      case 6: hipLaunchKernelGGL((adj_brick_kernel<6, false>), grid, block, 0, st, a); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  const bool xyp = (a.g.bc[0] == BC_PERIODIC && a.g.bc[1] == BC_PERIODIC);
  return xyp ? launch_field_x<true>(s, seed, a, st) : launch_field_x<false>(s, seed, a, st);
}

hipError_t launch_adj_gather(const AdjArgs& a, int mode, int stage, hipStream_t st) {
  const int bxs = (a.g.n[0] + 63) / 64, bys = (a.g.n[1] + 3) / 4;
  const long long blocks = (long long)bxs * bys * a.g.n[2];
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  switch (mode == 0 ? stage : 10 + mode) {
    case 2: hipLaunchKernelGGL((adj_gather_kernel<0, 2>), grid, block, 0, st, a, bxs, bys); break;
    case 3: hipLaunchKernelGGL((adj_gather_kernel<0, 3>), grid, block, 0, st, a, bxs, bys); break;
    case 4: hipLaunchKernelGGL((adj_gather_kernel<0, 4>), grid, block, 0, st, a, bxs, bys); break;
    case 5: hipLaunchKernelGGL((adj_gather_kernel<0, 5>), grid, block, 0, st, a, bxs, bys); break;
    case 6: hipLaunchKernelGGL((adj_gather_kernel<0, 6>), grid, block, 0, st, a, bxs, bys); break;
    case 11: hipLaunchKernelGGL((adj_gather_kernel<1, 1>), grid, block, 0, st, a, bxs, bys); break;
    case 12: hipLaunchKernelGGL((adj_gather_kernel<2, 1>), grid, block, 0, st, a, bxs, bys); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fill(double* v, long long n, double val, hipStream_t st) {
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(256), 0, st, v, n, val);
  return hipGetLastError();
}

hipError_t launch_seg_step(Control* c2, const double* dt_record, long long n, hipStream_t st) {
  hipLaunchKernelGGL(seg_step_kernel, dim3(1), dim3(64), 0, st, c2, dt_record, n);
  return hipGetLastError();
}

}  // namespace relax
