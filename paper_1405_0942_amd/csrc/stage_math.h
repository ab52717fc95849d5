// stage_math.h -- the node-wise arithmetic of a Runge-Kutta stage, shared by the sweeps of stage.hip
// (z-marching tiles) and brick.hip (small grids): the current from F' and the differences of B or from
// the octilateral loops, the stage updates, the convexity test and the workgroup reductions.  In FP64 with
// the nearest-neighbour current a node's result does not depend on the sweep, bit for bit: the products
// are fused by hand, below.  FP32-mixed and the octilateral current leave that to the compiler, and may
// part by a rounding.  The method and the stored vectors are described at the top of stage.hip.  Internal
// to the library.
#pragma once

#include <type_traits>

#include "sweep_common.h"

namespace relax {

// What a stage reads and stores (S: stage 1..6; the variants are described at stage_kernel).
template <int S, bool MIXED, bool NNN>
struct Stage {
  using T = typename std::conditional<MIXED, float, double>::type;
  static constexpr bool STAGE1 = (S == 1);
  static constexpr bool LAST = (S == 6);
  static constexpr bool LEAN = !MIXED && !NNN;  // the lean set of stored vectors (above)
  // the window is a base vector (x_n; y_3 in stage 3, y_5 in stage 5) plus at most one vector
  // v with coefficient cv: k_1 (cv = dt a_21) in stage 2, d_4 and d_6 (cv = 1) in stages 4, 6
  static constexpr bool WV = (S == 2 || S == 4 || LAST);
  // own-node values carried from the window to the output node (3 planes later): x_n in
  // stages 2, 4, 6 (and k_1 in stage 2)
  static constexpr bool CX = WV;
  static constexpr bool CV = LEAN ? WV : (S == 2);
  // vectors read at the output node: lean, c_4 in stage 3 and k_1, k_3 in stage 4; else k_1, k_2
  // and k_1..k_3
  static constexpr int NPK = (S == 3) ? (LEAN ? 1 : 2) : (S == 4 ? (LEAN ? 2 : 3) : 0);
  static constexpr int NPKA = NPK > 0 ? NPK : 1;
  static constexpr bool PS = (S == 5 || LAST);             // partial sums read at the output node
  static constexpr int NPS = PS ? (LEAN && S == 5 ? 1 : 2) : 1;
  static constexpr bool SUMS_OUT = (S == 3 || S == 4 || S == 5);
};

// the outputs of one node
template <int S, bool MIXED, bool NNN, bool DIAG, bool REC>
struct StageOut {
  using T = typename Stage<S, MIXED, NNN>::T;
  T k[3];                                              // k_s (stages 1..3; stage 2: C4), u (DIAG)
  double y[3];                                         // x_n copy (stage 1), y_3 (stage 2), y_5 (stage 4), x_{n+1}
  T s[Stage<S, MIXED, NNN>::SUMS_OUT ? 3 : 1][3];      // stage 3: d_4; stage 4: P6, X, E; stage 5: P6, -, E
  double p[DIAG ? 3 : 1][3];                           // DIAG: B, J, alpha*
  double yc[REC && !DIAG ? 3 : 1];                              // REC: the stage input at the node
};

// the octilateral loops of Sec. 2.3 through the eight ring neighbours of each grid
// plane, taken literally: vertices V1..V8 = +a, +a+b, +b, -a+b, -a, -a-b, -b, +a-b;
// circulation sum (B_r + B_r+1)/2 . dx_r; area vector = the triangles at the edge
// points (V2 V3 V4, V4 V5 V6, V6 V7 V8, V8 V1 V2) plus the quadrilateral through the
// diagonal points V2 V4 V6 V8; then J . N_q = C_q by Cramer's rule
// pos, field: component m of x and B at the neighbour (dx, dy, dz)
template <typename Pos, typename Field>
__device__ __forceinline__ void octilateral(Pos pos, Field field, double J[3]) {
  constexpr int RD[9][2] = {{1, 0}, {1, 1}, {0, 1}, {-1, 1}, {-1, 0}, {-1, -1}, {0, -1}, {1, -1}, {1, 0}};
  double Mq[3][3], Cq[3];
#pragma unroll 1
  for (int qa = 0; qa < 3; qa++) {
    // (a, b) = (y, z), (z, x), (x, y); walk V1..V8 and back to V1, keeping only the
    // previous vertex, the previous edge and the diagonal points met so far
    double Vp[3], Bvp[3], ep[3], e1[3], D1[3], Dp[3], q1[3], qp[3];
    double circ = 0.0, nA[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r <= 8; r++) {
      const int da = RD[r][0], db = RD[r][1];
      const int dx = qa == 2 ? da : (qa == 1 ? db : 0);
      const int dy = qa == 0 ? da : (qa == 2 ? db : 0);
      const int dz = qa == 0 ? db : (qa == 1 ? da : 0);
      double V[3], Bv[3];
#pragma unroll
      for (int m = 0; m < 3; m++) {
        V[m] = pos(dx, dy, dz, m);
        Bv[m] = field(dx, dy, dz, m);
      }
      if (r > 0) {
        double e[3];
#pragma unroll
        for (int m = 0; m < 3; m++) {
          e[m] = V[m] - Vp[m];  // dx_r (1-based r), from V_r to V_r+1
          circ += 0.5 * (Bvp[m] + Bv[m]) * e[m];
        }
        // triangles at the edge points: dx2 x dx3, dx4 x dx5, dx6 x dx7 and dx8 x dx1
        if (r == 3 || r == 5 || r == 7) {
          nA[0] += 0.5 * (ep[1] * e[2] - ep[2] * e[1]);
          nA[1] += 0.5 * (ep[2] * e[0] - ep[0] * e[2]);
          nA[2] += 0.5 * (ep[0] * e[1] - ep[1] * e[0]);
        }
        if (r == 8) {
          nA[0] += 0.5 * (e[1] * e1[2] - e[2] * e1[1]);
          nA[1] += 0.5 * (e[2] * e1[0] - e[0] * e1[2]);
          nA[2] += 0.5 * (e[0] * e1[1] - e[1] * e1[0]);
        }
#pragma unroll
        for (int m = 0; m < 3; m++) {
          if (r == 1) e1[m] = e[m];
          ep[m] = e[m];
        }
      }
      // the quadrilateral through the diagonal points V2, V4, V6, V8 (r = 1, 3, 5, 7):
      // edges dx_A..dx_D and the sum of their consecutive cross products over 4
      if (r == 1 || r == 3 || r == 5 || r == 7) {
        if (r == 1) {
#pragma unroll
          for (int m = 0; m < 3; m++) D1[m] = V[m];
        } else {
          double qe[3];
#pragma unroll
          for (int m = 0; m < 3; m++) qe[m] = V[m] - Dp[m];
          if (r == 3) {
#pragma unroll
            for (int m = 0; m < 3; m++) q1[m] = qe[m];
          } else {
            nA[0] += 0.25 * (qp[1] * qe[2] - qp[2] * qe[1]);
            nA[1] += 0.25 * (qp[2] * qe[0] - qp[0] * qe[2]);
            nA[2] += 0.25 * (qp[0] * qe[1] - qp[1] * qe[0]);
          }
#pragma unroll
          for (int m = 0; m < 3; m++) qp[m] = qe[m];
          if (r == 7) {  // the closing edge V8 -> V2, then its products with dx_C and dx_A
            double qd[3];
#pragma unroll
            for (int m = 0; m < 3; m++) qd[m] = D1[m] - V[m];
            nA[0] += 0.25 * (qe[1] * qd[2] - qe[2] * qd[1]) + 0.25 * (qd[1] * q1[2] - qd[2] * q1[1]);
            nA[1] += 0.25 * (qe[2] * qd[0] - qe[0] * qd[2]) + 0.25 * (qd[2] * q1[0] - qd[0] * q1[2]);
            nA[2] += 0.25 * (qe[0] * qd[1] - qe[1] * qd[0]) + 0.25 * (qd[0] * q1[1] - qd[1] * q1[0]);
          }
        }
#pragma unroll
        for (int m = 0; m < 3; m++) Dp[m] = V[m];
      }
#pragma unroll
      for (int m = 0; m < 3; m++) {
        Vp[m] = V[m];
        Bvp[m] = Bv[m];
      }
    }
#pragma unroll
    for (int m = 0; m < 3; m++) Mq[qa][m] = nA[m];
    Cq[qa] = circ;
  }
  const double iM = 1.0 / det3(Mq);
#pragma unroll
  for (int c = 0; c < 3; c++) {
    double Mc[3][3];
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
      for (int k = 0; k < 3; k++) Mc[r][k] = (k == c) ? Cq[r] : Mq[r][k];
    J[c] = det3(Mc) * iM;
  }
}

// The products of the FP64 nearest-neighbour path with every fused multiply-add written out: left to
// the compiler, the same expression may be fused in different orders in the march and in the bricks,
// and a node's result would then depend on the sweep in its last bit.
__device__ __forceinline__ double dot3(double a0, double b0, double a1, double b1, double a2, double b2) {
  return fma(a2, b2, fma(a0, b0, a1 * b1));
}
__device__ __forceinline__ double minor2(double a, double b, double c, double d) {  // a b - c d
  const double cd = c * d;
  return fma(a, b, -cd);
}
__device__ __forceinline__ double det3_fused(const double F[3][3]) {
  const double s = F[0][1] * minor2(F[1][0], F[2][2], F[1][2], F[2][0]);
  return fma(F[0][2], minor2(F[1][0], F[2][1], F[1][1], F[2][0]),
             fma(F[0][0], minor2(F[1][1], F[2][2], F[1][2], F[2][1]), -s));
}

// J = F' c' / det F' from the differences G'[a][m] = B_m(n + e_a) - B_m(n - e_a), with
// c'_q = (F' e_b) . G'_a - (F' e_a) . G'_b, (a, b, q) = (y, z, x), (z, x, y), (x, y, z)
__device__ __forceinline__ void current(const double F[3][3], const double G[3][3], double rD, double J[3]) {
#pragma clang fp contract(off)
  double cq[3];
#pragma unroll
  for (int q = 0; q < 3; q++) {
    const int a = (q + 1) % 3, b = (q + 2) % 3;
    cq[q] = dot3(F[0][b], G[a][0], F[1][b], G[a][1], F[2][b], G[a][2]) -
            dot3(F[0][a], G[b][0], F[1][a], G[b][1], F[2][a], G[b][2]);
  }
#pragma unroll
  for (int m = 0; m < 3; m++) J[m] = dot3(F[m][0], cq[0], F[m][1], cq[1], F[m][2], cq[2]) * rD;
}
__device__ __forceinline__ void current(const float F[3][3], const float G[3][3], float rD, float J[3]) {
  float cq[3];
  cq[0] = F[0][2] * G[1][0] + F[1][2] * G[1][1] + F[2][2] * G[1][2] -
          (F[0][1] * G[2][0] + F[1][1] * G[2][1] + F[2][1] * G[2][2]);
  cq[1] = F[0][0] * G[2][0] + F[1][0] * G[2][1] + F[2][0] * G[2][2] -
          (F[0][2] * G[0][0] + F[1][2] * G[0][1] + F[2][2] * G[0][2]);
  cq[2] = F[0][1] * G[0][0] + F[1][1] * G[0][1] + F[2][1] * G[0][2] -
          (F[0][0] * G[1][0] + F[1][0] * G[1][1] + F[2][0] * G[1][2]);
#pragma unroll
  for (int m = 0; m < 3; m++) J[m] = (F[m][0] * cq[0] + F[m][1] * cq[1] + F[m][2] * cq[2]) * rD;
}

// f = J x B
template <bool NNN, typename T>
__device__ __forceinline__ void force(const T J[3], const T B[3], T f[3]) {
#pragma unroll
  for (int m = 0; m < 3; m++) {
    const int a = (m + 1) % 3, b = (m + 2) % 3;
    if constexpr (!NNN && sizeof(T) == 8)
      f[m] = minor2(J[a], B[b], J[b], B[a]);
    else
      f[m] = J[a] * B[b] - J[b] * B[a];
  }
}

// B = F' B0'' / det F'
template <typename T>
__device__ __forceinline__ void pull_back(const double F[3][3], T q0, T q1, T q2, double rD, T B[3]) {
  if constexpr (sizeof(T) == 4) {
    const float fi = (float)rD;
#pragma unroll
    for (int m = 0; m < 3; m++)
      B[m] = ((float)F[m][0] * q0 + (float)F[m][1] * q1 + (float)F[m][2] * q2) * fi;
  } else {
#pragma unroll
    for (int m = 0; m < 3; m++) B[m] = dot3(F[m][0], q0, F[m][1], q1, F[m][2], q2) * rD;
  }
}

// Convexity (Sec. 3.2.3, eq. "convexity"): every trihedron of edge vectors to the neighbours
// p + di e_x, p + dj e_y, p + dk e_z ([0]: toward -, [1]: toward +) must have a determinant of sign
// di dj dk; trihedra beyond a line-tied face are not formed.
__device__ __forceinline__ bool is_convex(const double ex[2][3], const double ey[2][3], const double ez[2][3], bool lox,
                                          bool hix, bool loy, bool hiy, bool loz, bool hiz) {
  bool convex = true;
#pragma unroll
  for (int t = 0; t < 8; t++) {
    const int a = t & 1, b = (t >> 1) & 1, c = (t >> 2) & 1;
    const bool formed = (a ? hix : lox) && (b ? hiy : loy) && (c ? hiz : loz);
    const double* u1 = ex[a];
    const double* u2 = ey[b];
    const double* u3 = ez[c];
    const double det = u1[0] * (u2[1] * u3[2] - u2[2] * u3[1]) - u1[1] * (u2[0] * u3[2] - u2[2] * u3[0]) +
                       u1[2] * (u2[0] * u3[1] - u2[1] * u3[0]);
    const double want = ((a + b + c) & 1) ? 1.0 : -1.0;  // (2a-1)(2b-1)(2c-1)
    if (formed && !(det * want > 0.0)) convex = false;
  }
  return convex;
}

// the reductions of a thread's nodes
struct Sums {
  double E = 0.0, R2 = 0.0, min_det = INFINITY, nulls = 0.0, concave = 0.0, lam = 0.0;
  // xi: the node of largest |f|^2 / B^4 so far, kept as (|f|^2, B^4, B^2) and compared by
  // cross-multiplication, so that the square root and the division are taken once at the end
  double xi_F2 = 0.0, xi_B4 = 1.0, xi_B2 = 1.0;

  __device__ __forceinline__ void force(double F2, double B2, double D, double tau_B2) {
    R2 += D * F2;
    if (B2 > tau_B2) {
      const double B4 = B2 * B2;
      if (F2 * xi_B4 > xi_F2 * B4 || F2 != F2) {
        xi_F2 = F2;
        xi_B4 = B4;
        xi_B2 = B2;
      }
    } else {
      nulls += 1.0;
    }
  }
  __device__ __forceinline__ void error(double err) { lam = (err > lam || err != err) ? err : lam; }
};

// Workgroup reductions of NT threads, in a fixed order, into the partial record of stage 1 ...
template <int NT, bool DIAG>
__device__ __forceinline__ void store_sums(const Sums& c, double red[NT / 64][NPART], double* pp) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const double e = wave_sum(c.E), r2 = wave_sum(c.R2), xi = wave_max(sqrt(c.xi_F2) / c.xi_B2),
               mn = wave_min(c.min_det), nl = wave_sum(c.nulls), cc = DIAG ? wave_sum(c.concave) : 0.0;
  if (lane == 63) {
    red[wave][0] = e;
    red[wave][1] = r2;
    red[wave][2] = xi;
    red[wave][3] = mn;
    red[wave][4] = nl;
    red[wave][5] = cc;
  }
  __syncthreads();
  if (tid < 6) {  // a thread per quantity
    double sum = 0, X = 0, M = INFINITY;
#pragma unroll
    for (int w = 0; w < NT / 64; w++) {
      const double v = red[w][tid];
      sum += v;
      X = max_nan(X, v);
      M = min_nan(M, v);
    }
    pp[tid] = tid == 2 ? X : (tid == 3 ? M : sum);
  }
}

// ... and into the Lambda partial of stage 6
template <int NT>
__device__ __forceinline__ void store_lambda(const Sums& c, double red[NT / 64][NPART], double* pl) {
  const int tid = threadIdx.x;
  const double l = wave_max(c.lam);
  if ((tid & 63) == 63) red[tid >> 6][6] = l;
  __syncthreads();
  if (tid == 0) {
    double L = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; w++) L = max_nan(L, red[w][6]);
    *pl = L;
  }
}

// The updates of stages 2..6 at one node from u = k_s, the own node's x_n and window vector v, and the
// vectors read at the node (pk: the k_j, or C4; ps: the partial sums).  Stage 6: err = |x5 - x4|.
template <int S, bool MIXED, bool NNN, bool REC, typename T = typename Stage<S, MIXED, NNN>::T>
__device__ __forceinline__ void advance(const T u[3], const double xq[3], const T vq[3], const T (*pk)[3],
                                        const T (*ps)[3], double dt, StageOut<S, MIXED, NNN, false, REC>& so,
                                        double err[3]) {
  constexpr bool LEAN = Stage<S, MIXED, NNN>::LEAN;
  constexpr int NPKA = Stage<S, MIXED, NNN>::NPKA, NPS = Stage<S, MIXED, NNN>::NPS;
  if constexpr (S == 2) {
    // y_3 = x_n + dt (a_31 k_1 + a_32 k_2), from the own node's x_n and k_1 of plane q
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const double d3 = fma(dt * CK::a[2][1], (double)u[m], (dt * CK::a[2][0]) * (double)vq[m]);
      so.y[m] = xq[m] + d3;
      if constexpr (LEAN)
        so.k[m] = fma(dt * CK::a[3][1], u[m], (dt * CK::a[3][0]) * vq[m]);
      else
        so.k[m] = u[m];
    }
  } else if constexpr (S == 3) {
    // d_4 = dt (a_41 k_1 + a_42 k_2 + a_43 k_3)
#pragma unroll
    for (int m = 0; m < 3; m++) {
      double d4 = (double)pk[0][m];
      if constexpr (!LEAN) {
        d4 = (dt * CK::a[3][0]) * (double)pk[0][m];
        d4 = fma(dt * CK::a[3][1], (double)pk[NPKA - 1][m], d4);
      }
      d4 = fma(dt * CK::a[3][2], (double)u[m], d4);
      so.k[m] = u[m];
      so.s[0][m] = (T)d4;
    }
  } else if constexpr (S == 4) {
    // y_5 = x_n + d_5, and the partial sums of k_1..k_4 the last two stages need
    // (b5_2 = b4_2 = 0: k_2 enters neither X nor E)
    if constexpr (LEAN) {
      // dt a_42 k_2 = d_4 - dt a_41 k_1 - dt a_43 k_3, from the own node's d_4
      constexpr double r5 = CK::a[4][1] / CK::a[3][1], r6 = CK::a[5][1] / CK::a[3][1];
      // E is stored less the multiple of P6 that stage 6 adds back as d_6 = P6 + dt a_65 k_5
      constexpr double mu = CK::e[4] / CK::a[5][4];
#pragma unroll
      for (int m = 0; m < 3; m++) {
        const double k1 = pk[0][m], k3 = pk[1][m], k4 = u[m], d4 = vq[m];
        double d5 = r5 * d4;
        d5 = fma(dt * (CK::a[4][0] - r5 * CK::a[3][0]), k1, d5);
        d5 = fma(dt * (CK::a[4][2] - r5 * CK::a[3][2]), k3, d5);
        d5 = fma(dt * CK::a[4][3], k4, d5);
        double p6 = r6 * d4;
        p6 = fma(dt * (CK::a[5][0] - r6 * CK::a[3][0]), k1, p6);
        p6 = fma(dt * (CK::a[5][2] - r6 * CK::a[3][2]), k3, p6);
        p6 = fma(dt * CK::a[5][3], k4, p6);
        double xs = (dt * CK::b5[0]) * k1;
        xs = fma(dt * CK::b5[2], k3, xs);
        xs = fma(dt * CK::b5[3], k4, xs);
        double es = -mu * p6;
        es = fma(dt * CK::e[0], k1, es);
        es = fma(dt * CK::e[2], k3, es);
        es = fma(dt * CK::e[3], k4, es);
        so.y[m] = xq[m] + d5;
        so.s[0][m] = p6;
        so.s[1][m] = xs;
        so.s[2][m] = es;
      }
    } else {
#pragma unroll
      for (int m = 0; m < 3; m++) {
        const double k1 = pk[0][m], k2 = pk[1][m], k3 = pk[2][m], k4 = u[m];
        double d5 = (dt * CK::a[4][0]) * k1;
        d5 = fma(dt * CK::a[4][1], k2, d5);
        d5 = fma(dt * CK::a[4][2], k3, d5);
        d5 = fma(dt * CK::a[4][3], k4, d5);
        double p6 = (dt * CK::a[5][0]) * k1;
        p6 = fma(dt * CK::a[5][1], k2, p6);
        p6 = fma(dt * CK::a[5][2], k3, p6);
        p6 = fma(dt * CK::a[5][3], k4, p6);
        double xs = (dt * CK::b5[0]) * k1;
        xs = fma(dt * CK::b5[2], k3, xs);
        xs = fma(dt * CK::b5[3], k4, xs);
        double es = (dt * (CK::b5[0] - CK::b4[0])) * k1;
        es = fma(dt * (CK::b5[2] - CK::b4[2]), k3, es);
        es = fma(dt * (CK::b5[3] - CK::b4[3]), k4, es);
        so.y[m] = xq[m] + d5;
        so.s[0][m] = (T)p6;
        so.s[1][m] = (T)xs;
        so.s[2][m] = (T)es;
      }
    }
  } else if constexpr (S == 5) {
#pragma unroll
    for (int m = 0; m < 3; m++) {
      so.s[0][m] = (T)fma(dt * CK::a[5][4], (double)u[m], (double)ps[0][m]);
      if constexpr (!LEAN) so.s[2][m] = (T)fma(dt * (CK::b5[4] - CK::b4[4]), (double)u[m], (double)ps[NPS - 1][m]);
    }
  } else {
    // x_{n+1} = x_n + (X + dt b5_6 k_6);  error E + dt (b5_6 - b4_6) k_6
#pragma unroll
    for (int m = 0; m < 3; m++) {
      so.y[m] = xq[m] + fma(dt * CK::b5[5], (double)u[m], (double)ps[0][m]);
      double es = (double)ps[NPS - 1][m];
      if constexpr (LEAN) es = fma(CK::e[4] / CK::a[5][4], vq[m], es);
      const double e = fma(dt * (CK::b5[5] - CK::b4[5]), (double)u[m], es);
      err[m] = fabs(e);
    }
  }
}

}  // namespace relax
