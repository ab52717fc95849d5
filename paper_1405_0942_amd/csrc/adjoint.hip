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
// The stage-6 field sweep scales xbar_{n+1} itself; the gather of stage t writes ybar_t (or sums of
// them) and kbar_{t-1}, which the field sweep of stage t - 1 reads.
//
// Seeds (seed mode of adj_field_kernel): E_M = 1/2 sum zeta |B|^2 det F dV adds kappa D' B to
// Bbar and 1/2 kappa |B|^2 to Dbar' (kappa = zeta dV / (8 hx hy hz)); R2 = 1/2 sum_interior
// det F |f|^2 dV enters through ubar = det F dV f / gamma (read from a buffer) plus
// 1/2 |f|^2 dV / (8 hx hy hz) on Dbar'.
//
// The field sweep is laid out like the forward stage sweep, with one barrier per plane step: a 64 x 8
// tile marching up a z-chunk, the stage input in an LDS ring of four planes (stages 3..6 stencil the
// stored y_s of the step), B and Gbar'_y in LDS by parity of the plane.  Gbar'_x needs none: a wave is
// a row of the tile, so its lanes hand it on, and only the columns beside the tile go through LDS.  The
// in-plane sums of plane p are taken after its barrier and kept in registers, where the transpose of
// plane p - 1 finds all it needs one step later.  The sums of the one-sided rows beyond line-tied faces (see stage.hip) give every node
// the same path.  Loads and stores are those of buffer instructions with masked-off lanes (offsets
// past the record count), issued one plane step ahead, so no divergent branch surrounds a memory
// instruction and the waits are exact.
//
// What bounds it: 64 x 64 x 192, 256 chunks of 6 planes, 45 us a sweep (46 with two barriers and three
// planes, 58 -> 50 at stage 2): 24 vectors with their halos at 4.6 TB/s through L2.  us per step of a
// backward pass over 128^3 periodic 1579 -> 1518, 129^3 line-tied 2373 -> 2041 (one-sided rows had
// diverged), 73 x 73 x 200 line-tied 1487 -> 1219.
#include "brick.h"
#include "tile.h"

#include <algorithm>

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
  if (!SEED || interior) {  // ub = 0 on a face, and every term but the seed's has that factor
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

// The neighbour's value along a wave, whose lanes are one row of the tile: from the lane below (UP false)
// or above; the end lane, which has no neighbour, gets `edge`.
template <bool UP>
__device__ __forceinline__ double neighbour(double v, double edge) {
  const u32x2 a = __builtin_bit_cast(u32x2, v), e = __builtin_bit_cast(u32x2, edge);
  constexpr int CTRL = UP ? 0x130 : 0x138;  // wave_shl:1, wave_shr:1
  u32x2 r;
  r.x = __builtin_amdgcn_update_dpp(e.x, a.x, CTRL, 0xf, 0xf, false);
  r.y = __builtin_amdgcn_update_dpp(e.y, a.y, CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, r);
}

template <int S, bool SEED, int FACES>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void adj_field_kernel(AdjArgs a) {
  constexpr bool WK = (!SEED && S == 2);  // the window carries k_1 too
  constexpr int NP2 = (RY2 * RX2 + NTHREADS - 1) / NTHREADS;
  constexpr int NP1 = (RY1 * RX1 + NTHREADS - 1) / NTHREADS;
  constexpr int NPG = (6 * (RY2 + RX2) + NTHREADS - 1) / NTHREADS;
  static_assert(TX == 64 && NP1 == 2, "a wave is a row of the tile; at most one halo point per thread");

  const Geometry& g = a.g;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const long long N = g.N;
  const unsigned nxy = (unsigned)nx * (unsigned)ny;
  const int bcx = g.bc[0], bcy = g.bc[1], bcz = g.bc[2];
  const double gamma = a.gamma;

  const double dt = SEED ? 0.0 : *a.dt;
  const double c21 = dt * CK::a[1][0];
  // the cotangent of u: seed buffer, dt b5_6 xbar_{n+1} (stage 6), or the gathered kbar_s
  const bool v_on = !SEED || a.useed != nullptr;
  const double* __restrict__ vsrc = SEED ? (a.useed ? a.useed : a.B0) : (S == 6 ? a.xbar : a.ubar);
  const double cv = (!SEED && S == 6) ? dt * CK::b5[5] : 1.0;
  const double* __restrict__ wsrc = (SEED || S <= 2) ? a.x : a.y[S > 2 ? S - 3 : 0];
  const double* __restrict__ k1p = a.k1;

  const int lb = logical_block(blockIdx.x, g.nblocks);
  const int tile_x = lb % g.tiles[0];
  const int tile_y = (lb / g.tiles[0]) % g.tiles[1];
  const int chunk = lb / (g.tiles[0] * g.tiles[1]);
  const int i0 = tile_x * TX, j0 = tile_y * TY;
  const int z0 = chunk * g.tz;
  const int z1 = min(z0 + g.tz, nz);
  const int tid = threadIdx.x;
  const int tx = tid % TX, ty = tid / TX;

  __shared__ double ys[4][3][RY2 * RX2];  // stage input, ring of 4 planes
  __shared__ double bs[2][3][RY1 * RX1];  // B on the tile + 1 halo, by parity of the plane
  __shared__ double gy[2][3][RY1 * TX];   // Gbar'_y on the tile and the rows beside it
  __shared__ double gx[2][3][2][TY];      // Gbar'_x on the columns beside the tile

  auto zload = [&](int pz) {
    if (FACES == FACES_NONE || bcz == BC_PERIODIC) return resolve_near(pz, nz, BC_PERIODIC).i;
    return min(max(pz, 0), nz - 1);
  };

  // index tables (as in the forward sweep): window point and field point 0 of a thread are its tile node
  unsigned w2e[NP2];
  int w2w[NP2], w2o[NP2];
#pragma unroll
  for (int r = 0; r < NP2; r++) {
    const int e = tid + r * NTHREADS;
    int row, col;
    if (e < NTHREADS) {
      row = ty + 2;
      col = tx + 2;
    } else {
      const int e2 = e - NTHREADS;
      if (e2 < 4 * RX2) {
        const int band = e2 / RX2;
        row = band < 2 ? band : RY2 - 4 + band;
        col = e2 - band * RX2;
      } else {
        const int e3 = e2 - 4 * RX2, side = e3 & 3;
        row = 2 + (e3 >> 2);
        col = side < 2 ? side : RX2 - 4 + side;
      }
    }
    const bool in_win = e < RY2 * RX2;
    const AxisIdx rx = axis_index(i0 + col - 2, nx, bcx), ry = axis_index(j0 + row - 2, ny, bcy);
    w2e[r] = (in_win && rx.ok && ry.ok) ? (unsigned)(ry.i * nx + rx.i) : IE;
    w2w[r] = (ry.w << 16) + (rx.w & 0xffff);
    w2o[r] = in_win ? row * RX2 + col : -1;
  }
  // ---- loads, issued one plane step ahead of their use ---------------------------------------
  struct Window {
    double x[NP2][3];
    double k[WK ? NP2 : 1][3];
  };
  auto load_window = [&](Window& w, int pz, bool on) {
    const long long zo = (long long)zload(pz) * nxy;
    unsigned e[NP2];
#pragma unroll
    for (int r = 0; r < NP2; r++) e[r] = on ? w2e[r] : IE;
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const auto rs = plane_rsrc(wsrc + m * N + zo, nxy);
#pragma unroll
      for (int r = 0; r < NP2; r++) w.x[r][m] = bload<double>(rs, e[r]);
    }
    if constexpr (WK) {
#pragma unroll
      for (int m = 0; m < 3; m++) {
        const auto rs = plane_rsrc(k1p + m * N + zo, nxy);
#pragma unroll
        for (int r = 0; r < NP2; r++) w.k[r][m] = bload<double>(rs, e[r]);
      }
    }
  };
  const bool perz = FACES == FACES_NONE || bcz == BC_PERIODIC;
  const int pb0 = perz ? z0 - 1 : max(z0 - 1, 0);
  const int pb1 = perz ? z1 : min(z1, nz - 1);
  const int pw1 = perz ? pb1 + 1 : min(pb1 + 1, nz - 1);  // last plane of the stage input

  // the first three planes, so that the rest of the tables is built while they are under way (64 x 64 x 192:
  // 654 -> 634 us per step of a backward pass)
  const bool low = !perz && pb0 == 0;  // the plane below holds the sums of the face
  const int lo = low ? 0 : pb0 - 1;
  Window w0, w1, w2;
  load_window(w0, lo, true);
  load_window(w1, lo + 1, true);
  load_window(w2, lo + 2, true);
  __builtin_amdgcn_sched_barrier(0);

  unsigned f1e[NP1];
  int f1o[NP1];            // offset in the B window (-1: no point)
  int f1y[NP1];            // offset in the stage-input window
  int f1dx[NP1], f1dy[NP1];  // offsets of the two points whose difference is F' along x, along y: plus | minus << 16
  bool f1live[NP1];        // on the grid and not on a line-tied face across x or y
  int halo_row = 0, halo_col = 0;
#pragma unroll
  for (int r = 0; r < NP1; r++) {
    const int e = tid + r * NTHREADS;
    int r1, c1;
    if (e < NTHREADS) {
      r1 = ty + 1;
      c1 = tx + 1;
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
      halo_row = r1;
      halo_col = c1;
    }
    const bool in_win = e < RY1 * RX1;
    const AxisIdx rx = axis_index(i0 + c1 - 1, nx, bcx), ry = axis_index(j0 + r1 - 1, ny, bcy);
    f1e[r] = (in_win && rx.ok && ry.ok) ? (unsigned)(ry.i * nx + rx.i) : IE;
    f1o[r] = in_win ? r1 * RX1 + c1 : -1;
    int ends = 0;  // 1, 2: low, high end along x; 4, 8: along y
    if (bcx == BC_LINE_TIED) ends |= rx.i == 0 ? 1 : (rx.i == nx - 1 ? 2 : 0);
    if (bcy == BC_LINE_TIED) ends |= ry.i == 0 ? 4 : (ry.i == ny - 1 ? 8 : 0);
    f1y[r] = (r1 + 1) * RX2 + c1 + 1;
    f1dx[r] = difference_points(f1y[r], 1, ends & 3);
    f1dy[r] = difference_points(f1y[r], RX2, ends >> 2);
    f1live[r] = f1e[r] != IE && ends == 0;
  }
  // the sums of the rows of line-tied faces across x and y, just beyond them (see stage.hip)
  constexpr int NGC = 3 * RY2, NGR = 3 * RX2;
  int gh_o[NPG], gh_s[NPG];
#pragma unroll
  for (int r = 0; r < NPG; r++) {
    gh_o[r] = -1;
    gh_s[r] = 0;
    const int t = tid + r * NTHREADS;
    if (t < 2 * NGC) {
      const int side = t / NGC, t1 = t - side * NGC, m = t1 / RY2, row = t1 - m * RY2;
      const int col = side == 0 ? 1 - i0 : nx - i0 + 2;
      if (bcx == BC_LINE_TIED && col >= 0 && col < RX2) {
        gh_o[r] = m * (RY2 * RX2) + row * RX2 + col;
        gh_s[r] = side == 0 ? 1 : -1;
      }
    } else if (t < 2 * NGC + 2 * NGR) {
      const int t0 = t - 2 * NGC, side = t0 / NGR, t1 = t0 - side * NGR, m = t1 / RX2, col = t1 - m * RX2;
      const int row = side == 0 ? 1 - j0 : ny - j0 + 2;
      if (bcy == BC_LINE_TIED && row >= 0 && row < RY2) {
        gh_o[r] = m * (RY2 * RX2) + row * RX2 + col;
        gh_s[r] = side == 0 ? RX2 : -RX2;
      }
    }
  }
  const int gi_t = i0 + tx, gj_t = j0 + ty;
  const bool tile_ok = (gi_t < nx) && (gj_t < ny);
  const unsigned out_e = tile_ok ? (unsigned)(gj_t * nx + gi_t) : IE;

  double b0r[NP1][3], vr[NP1][3];
  double bbr[3];  // B0bar'' at the output node
  auto commit_window = [&](const Window& w, int pz) {
    const double shz = resolve_near(pz, nz, bcz).w * g.period[2];
    const int slot = pz & 3;
#pragma unroll
    for (int r = 0; r < NP2; r++) {
      double v[3];
#pragma unroll
      for (int m = 0; m < 3; m++) {
        v[m] = w.x[r][m];
        if constexpr (WK) v[m] = fma(c21, w.k[r][m], v[m]);
      }
      v[0] += (double)(short)(w2w[r] & 0xffff) * g.period[0];
      v[1] += (double)(w2w[r] >> 16) * g.period[1];
      v[2] += shz;
      if (w2o[r] >= 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) ys[slot][m][w2o[r]] = (w2e[r] != IE) ? v[m] : 0.0;
      }
    }
  };
  // the sums of a line-tied z face, in the plane beyond it, from the face's plane pa and the next, pb
  auto commit_sum_plane = [&](int pz, int pa, int pb) {
#pragma unroll
    for (int r = 0; r < NP2; r++) {
      if (w2o[r] >= 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) ys[pz & 3][m][w2o[r]] = face_sum(ys[pa & 3][m][w2o[r]], ys[pb & 3][m][w2o[r]]);
      }
    }
  };
  auto fill_sums = [&](int pz) {
    if constexpr (FACES != FACES_XY) return;
#pragma unroll
    for (int r = 0; r < NPG; r++) {
      if (gh_o[r] >= 0) {
        double* y = &ys[pz & 3][0][gh_o[r]];
        *y = face_sum(y[gh_s[r]], y[2 * gh_s[r]]);
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
  auto store_point = [&](const double Fb[9], const double B0b[3], int qz, bool on) {
    const long long zo = (long long)zload(qz) * nxy;
    const unsigned eo = on ? out_e : IE;
#pragma unroll
    for (int i = 0; i < 9; i++) bstore(plane_rsrc(a.Fbar + i * N + zo, nxy), eo, Fb[i]);
#pragma unroll
    for (int m = 0; m < 3; m++) bstore(plane_rsrc(a.B0bar + m * N + zo, nxy), eo, B0b[m]);
  };

  // ---- prologue: the stage input on the planes pb0 - 1 .. pb0 + 1
  Window win;
  {
    commit_window(w0, lo);
    commit_window(w1, lo + 1);
    commit_window(w2, lo + 2);
    if (low) commit_sum_plane(-1, 0, 1);  // plane 2 is committed again by the first plane step
  }
  __syncthreads();
  fill_sums(pb0);
  // leave the same loads and (dropped) stores in flight, in the same order, as a plane step
  load_window(win, pb0 + 2, pb0 + 2 <= pw1);
  load_field(pb0);
  load_point(pb0 - 1);
  {
    const double zero[9] = {};
    store_point(zero, zero, pb0 - 1, false);
  }
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();

  // own-node values carried between plane steps; q = p - 1 is the output plane
  double Fq[3][3] = {}, rDq = 0.0, ubq[3] = {}, b0q[3] = {};
  double Bq[3] = {}, Bqm[3] = {};    // B at q, q - 1
  double gzq[3] = {}, gzqm[3] = {};  // Gbar'_z at q, q - 1
  double Gq[2][3] = {};              // x and y differences of B at q
  double Btq[3] = {};                // in-plane transpose of Gbar' at q
  const int ot = (ty + 1) * RX1 + (tx + 1);

  for (int p = pb0; p <= z1; p++) {
    const int q = p - 1;
    const bool qout = (q >= z0 && q < z1);
    fill_sums(p + 1);
    // 1. commit the plane the next field needs, load the one after it
    if (perz || p + 2 < nz)  // past the chunk's last plane: zeros that nothing reads; beyond a face see stage.hip
      commit_window(win, p + 2);
    else if (p + 2 == nz)
      commit_sum_plane(nz, nz - 1, nz - 2);
    load_window(win, p + 3, p + 3 <= pw1);

    // 2. B and Gbar' of the field points of plane p, 0 off the grid
    const bool on_p = p <= pb1, live_p = on_p && (perz || (p > 0 && p < nz - 1));
    double F[3][3], rD, ub[3], B[3], Gx[3], Gy[3], Gz[3];
    // the planes whose difference is F' along z (line-tied faces: the sum and plane 2 or nz - 3)
    const bool low_face = !perz && p == 0, high_face = !perz && p == nz - 1;
    const int sp = (low_face ? -1 : (high_face ? p - 2 : p + 1)) & 3;
    const int sm = (low_face ? 2 : (high_face ? p + 1 : p - 1)) & 3;
    auto field = [&](auto point) {
      constexpr int R = decltype(point)::value;
      const int o = f1y[R];
      int dx = f1dx[R], dy = f1dy[R];
      if constexpr (FACES == FACES_XY) {  // taken apart here, not kept apart over the march: registers
        pin(dx);
        pin(dy);
      }
      const int sc = p & 3;
#pragma unroll
      for (int m = 0; m < 3; m++) {
        if constexpr (FACES == FACES_XY) {
          F[m][0] = ys[sc][m][dx & 0xffff] - ys[sc][m][dx >> 16];
          F[m][1] = ys[sc][m][dy & 0xffff] - ys[sc][m][dy >> 16];
        } else {
          F[m][0] = ys[sc][m][o + 1] - ys[sc][m][o - 1];
          F[m][1] = ys[sc][m][o + RX2] - ys[sc][m][o - RX2];
        }
        F[m][2] = ys[sp][m][o] - ys[sm][m][o];
      }
      const double r = rcp_nr(det3(F));
      rD = (on_p && f1e[R] != IE) ? r : 0.0;
#pragma unroll
      for (int m = 0; m < 3; m++) ub[m] = (live_p && f1live[R]) ? cv * vr[R][m] : 0.0;
      transpose_field(F, rD, b0r[R], ub, gamma, B, Gx, Gy, Gz);
#pragma unroll
      for (int m = 0; m < 3; m++) bs[p & 1][m][f1o[R]] = B[m];
    };
    if (f1o[1] >= 0) {
      field(std::integral_constant<int, 1>{});
      if (halo_row == 0 || halo_row == RY1 - 1) {
        if (halo_col >= 1 && halo_col <= TX) {
#pragma unroll
          for (int m = 0; m < 3; m++) gy[p & 1][m][halo_row * TX + halo_col - 1] = Gy[m];
        }
      } else {
#pragma unroll
        for (int m = 0; m < 3; m++) gx[p & 1][m][halo_col != 0][halo_row - 1] = Gx[m];
      }
    }
    field(std::integral_constant<int, 0>{});
#pragma unroll
    for (int m = 0; m < 3; m++) gy[p & 1][m][(ty + 1) * TX + tx] = Gy[m];
    double b0p[3];
#pragma unroll
    for (int m = 0; m < 3; m++) b0p[m] = b0r[0][m];
    load_field(min(p + 1, pb1));

    // 3. the transpose at the own node of plane q, from registers
    double Fb[9] = {}, B0b[3] = {};
    if (qout) {
      const bool face_q = !perz && (q == 0 || q == nz - 1);
      const bool interior = f1live[0] && !face_q;
      double G[3][3], Bt[3];  // Bt: sum_a Gbar'_a(m - e_a) - Gbar'_a(m + e_a)
#pragma unroll
      for (int m = 0; m < 3; m++) {
        G[0][m] = Gq[0][m];
        G[1][m] = Gq[1][m];
        G[2][m] = B[m] - Bqm[m];
        Bt[m] = Btq[m] + (gzqm[m] - Gz[m]);
      }
      double zeta = 1.0;
      if constexpr (SEED) {
        if (bcx == BC_LINE_TIED && (gi_t == 0 || gi_t == nx - 1)) zeta *= 0.5;
        if (bcy == BC_LINE_TIED && (gj_t == 0 || gj_t == ny - 1)) zeta *= 0.5;
        if (face_q) zeta *= 0.5;
      }
      double dB[3];
      transpose_node<SEED>(Fq, rDq, Bq, ubq, b0q, G, Bt, interior, zeta, a, Fb, dB);
#pragma unroll
      for (int m = 0; m < 3; m++) B0b[m] = bbr[m] + dB[m];
    }
    load_point(p);  // B0bar'' at the output node of the next plane step
    store_point(Fb, B0b, q, qout);
    __syncthreads();

    // 4. the in-plane part of the transpose at the own node of plane p, for the next step
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const double* b = bs[p & 1][m];
      const double* y = &gy[p & 1][m][(ty + 1) * TX + tx];
      Gq[0][m] = b[ot + 1] - b[ot - 1];
      Gq[1][m] = b[ot + RX1] - b[ot - RX1];
      const double below = neighbour<false>(Gx[m], gx[p & 1][m][0][ty]);
      const double above = neighbour<true>(Gx[m], gx[p & 1][m][1][ty]);
      Btq[m] = (below - above) + (y[-TX] - y[TX]);
      Bqm[m] = Bq[m];
      Bq[m] = B[m];
      gzqm[m] = gzq[m];
      gzq[m] = Gz[m];
      ubq[m] = ub[m];
      b0q[m] = b0p[m];
#pragma unroll
      for (int c = 0; c < 3; c++) Fq[m][c] = F[m][c];
    }
    rDq = rD;
  }
}

// The same for small grids, a brick of nodes per workgroup (see brick.hip): the stage input with its
// 2-node halo, B and the three Gbar' on the brick and its 1-node halo, all planes at once, two
// barriers.  LDS: up to 157 KB (Gbar' takes 72 bytes a field point), one workgroup per CU.  Up to
// 2^19 nodes (make_adj_geometry): us per step of a backward pass, march / bricks (its forward replay too):
// 65^3 line-tied 491 / 377, 73^3 line-tied 585 / 485, 80^3 periodic 581 / 512, 81^3 line-tied 652 / 621,
// 56 x 56 x 168 521 / 562, 90^3 periodic 772 / 748, 64 x 64 x 192 632 / 734.
constexpr int NPW = (ADJ_WINDOW + BRICK_THREADS - 1) / BRICK_THREADS;
constexpr int NPF = 1 + (BRICK_SHELL + BRICK_THREADS - 1) / BRICK_THREADS;

template <int S, bool SEED>
__global__ __launch_bounds__(BRICK_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void adj_brick_kernel(AdjArgs a) {
  constexpr bool WK = (!SEED && S == 2);
  const Geometry& g = a.g;
  const long long N = g.N;
  const Brick br(g);
  const BrickOrigin at0(br, g);
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

  // ---- all loads first; a wave skips the points past the brick's
  double wx[NPW][3], wk[WK ? NPW : 1][3];
  BrickPoint wp[NPW];
#pragma unroll
  for (int r = 0; r < NPW; r++) {
    const int e = tid + r * BRICK_THREADS;
    if (e < br.nwin) {
      wp[r] = brick_window(br, g, e, at0);
      const unsigned i = wp[r].index;
#pragma unroll
      for (int m = 0; m < 3; m++) wx[r][m] = at(wsrc + m * N, i);
      if constexpr (WK) {
#pragma unroll
        for (int m = 0; m < 3; m++) wk[r][m] = at(a.k1 + m * N, i);
      }
    }
  }
  double b0r[NPF][3], vr[NPF][3];
  BrickField fp[NPF];
#pragma unroll
  for (int r = 0; r < NPF; r++) {
    fp[r].slot = -1;
    if (r == 0 || tid + (r - 1) * BRICK_THREADS < br.nshell) {
      fp[r] = brick_field(br, g, r, tid, at0);
      const unsigned i = fp[r].index;
#pragma unroll
      for (int m = 0; m < 3; m++) {
        b0r[r][m] = at(a.B0 + m * N, i);
        vr[r][m] = at(vsrc + m * N, i);
      }
    }
  }
  const bool node = fp[0].node();
  const int own = fp[0].index;
  double bbr[3];
#pragma unroll
  for (int m = 0; m < 3; m++) bbr[m] = at(a.B0bar + m * N, (unsigned)own);
  const bool at_face = br.at_face(g, at0.i0, at0.j0, at0.k0);

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

  // ---- B and Gbar' on the brick and its 1-node halo
  double Fq[3][3], Bq[3], ubq[3], rDq;
#pragma unroll
  for (int r = 0; r < NPF; r++) {
    if (r == 0 || fp[r].slot >= 0) {
      const int o = fp[r].window;
      double F[3][3], B[3], Gx[3], Gy[3], Gz[3], ub[3];
      face_differences(br, fp[r].ends, at_face, ys, o, F);
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
// MODE 0 (stage STAGE >= 2): the cotangent of k_{t-1},
//   dt (b5_{t-1} xbar + sum_{t' >= t} a_{t',t-1} ybar_{t'}) -> ubar_out.
// MODE 1 (stage 1): xbar + D^T Fbar' + sum_{t=2..6} ybar_t -> xbar.  MODE 2 (seed): xbar = D^T Fbar'.
// Stages 6 and 5 store ybar_t.  Stage 4 stores, in place of ybar_6, ybar_5 and its own, what is still
// wanted of the three and of xbar: sum[0] = P2 = a62 ybar_6 + a52 ybar_5 + a42 ybar_4 for k_2 (b5_2 = 0),
// sum[1] = P1, likewise with b5_1 xbar, for k_1, and sum[2] = xbar + ybar_6 + ybar_5 + ybar_4.  That is
// 1008 instead of 1200 bytes a node and step for the six gathers, which bound them (64 x 64 x 192: 4.6 to
// 5.8 TB/s, 161 -> 153 us the six).
// One thread a node, rows of 64 along x so that every access is coalesced and no index needs a 64-bit
// division (16^3: 8 -> 4 us against a grid-stride loop with 64-bit divisions).  A launch takes the workgroups
// first, first + 1, ... of the pass: fewer than 2^32 work-items, which long thin grids pass (4 x 5 x 2^23).
template <int MODE, int STAGE>
__global__ __launch_bounds__(256) void adj_gather_kernel(AdjArgs a, int bxs, int bys, unsigned first) {
  const Geometry& g = a.g;
  const long long N = g.N;
  const int nx = g.n[0], ny = g.n[1];
  const int lb = (int)first + logical_block(blockIdx.x, gridDim.x);
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
    const long long o = p + r * N;
    if constexpr (MODE == 0) {
      constexpr int s = STAGE - 1;  // the stage whose k's cotangent is assembled
      const double y = yb[r];
      double v = CK::a[STAGE - 1][s - 1] * y;
      if constexpr (STAGE >= 4) {
        const double y5 = STAGE == 4 ? a.ybar[5][o] : 0.0;
        const double y6 = STAGE <= 5 ? a.ybar[6][o] : 0.0;
        const double x = STAGE <= 5 ? a.xbar[o] : 0.0;
        if constexpr (STAGE == 4) {
          v = CK::a[5][2] * y6 + CK::a[4][2] * y5 + v;
          a.sum[0][o] = CK::a[5][1] * y6 + CK::a[4][1] * y5 + CK::a[3][1] * y;
          a.sum[1][o] = CK::b5[0] * x + CK::a[5][0] * y6 + CK::a[4][0] * y5 + CK::a[3][0] * y;
          a.sum[2][o] = x + y6 + y5 + y;
        } else {
          if constexpr (STAGE == 5) v = CK::a[5][3] * y6 + v;
          a.ybar[STAGE][o] = y;
        }
        if constexpr (STAGE <= 5) v = CK::b5[s - 1] * x + v;  // b5_5 = 0
      } else if constexpr (STAGE == 3) {
        v = a.sum[0][o] + v;
        a.ybar[3][o] = y;
      } else {
        v = a.sum[1][o] + CK::a[2][0] * a.ybar[3][o] + v;
        a.ybar[2][o] = y;
      }
      a.ubar_out[o] = dt * v;
    } else if constexpr (MODE == 1) {
      a.xbar_out[o] = a.sum[2][o] + a.ybar[3][o] + a.ybar[2][o] + yb[r];
    } else {
      a.xbar_out[o] = yb[r];
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

template <int S, bool SEED>
hipError_t launch_field_t(const AdjArgs& a, hipStream_t st) {
  const dim3 grid(a.g.nblocks), block(NTHREADS);
  switch (faces_of(a.g)) {
    case FACES_NONE: hipLaunchKernelGGL((adj_field_kernel<S, SEED, FACES_NONE>), grid, block, 0, st, a); break;
    case FACES_Z: hipLaunchKernelGGL((adj_field_kernel<S, SEED, FACES_Z>), grid, block, 0, st, a); break;
    default: hipLaunchKernelGGL((adj_field_kernel<S, SEED, FACES_XY>), grid, block, 0, st, a); break;
  }
  return hipGetLastError();
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
  if (seed) return launch_field_t<1, true>(a, st);
  switch (s) {
    case 1: return launch_field_t<1, false>(a, st);
    case 2: return launch_field_t<2, false>(a, st);
    case 3: return launch_field_t<3, false>(a, st);
    case 4: return launch_field_t<4, false>(a, st);
    case 5: return launch_field_t<5, false>(a, st);
    case 6: return launch_field_t<6, false>(a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_adj_gather(const AdjArgs& a, int mode, int stage, hipStream_t st) {
  const int bxs = (a.g.n[0] + 63) / 64, bys = (a.g.n[1] + 3) / 4;
  const long long blocks = (long long)bxs * bys * a.g.n[2];
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  for (unsigned first = 0; first < (unsigned)blocks; first += GATHER_BLOCKS) {
    const dim3 grid(std::min<unsigned>(GATHER_BLOCKS, (unsigned)blocks - first)), block(256);
    switch (mode == 0 ? stage : 10 + mode) {
      case 2: hipLaunchKernelGGL((adj_gather_kernel<0, 2>), grid, block, 0, st, a, bxs, bys, first); break;
      case 3: hipLaunchKernelGGL((adj_gather_kernel<0, 3>), grid, block, 0, st, a, bxs, bys, first); break;
      case 4: hipLaunchKernelGGL((adj_gather_kernel<0, 4>), grid, block, 0, st, a, bxs, bys, first); break;
      case 5: hipLaunchKernelGGL((adj_gather_kernel<0, 5>), grid, block, 0, st, a, bxs, bys, first); break;
      case 6: hipLaunchKernelGGL((adj_gather_kernel<0, 6>), grid, block, 0, st, a, bxs, bys, first); break;
      case 11: hipLaunchKernelGGL((adj_gather_kernel<1, 1>), grid, block, 0, st, a, bxs, bys, first); break;
      case 12: hipLaunchKernelGGL((adj_gather_kernel<2, 1>), grid, block, 0, st, a, bxs, bys, first); break;
      default: return hipErrorInvalidValue;
    }
    if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
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
