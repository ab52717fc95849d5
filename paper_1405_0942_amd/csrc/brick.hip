// brick.hip -- the stage sweep for small grids: one workgroup per brick of nodes, all planes at once.
//
// The z-marching sweep of stage.hip pays one plane step after another: about 1.2 us of dependent FP64
// and LDS work each, with at least 12 steps per chunk, on a grid that has too few tiles to fill the
// CUs.  Here a workgroup of 512 threads loads the stage input of a whole brick with its 2-node halo
// into LDS at once, forms F', det F' and B on the brick and its 1-node halo (the own node first, then
// the shell), and the current, force and update of one node per thread: two barriers in all, so that a
// sweep takes one round of global latency instead of a dozen (16^3: 5.0 to 6.4 us a sweep, where
// the march took 42 to 57).  The price is the halo: a brick of 8 x 8 x 8 loads 3.4 window points and
// evaluates 2 fields per node where the march of a tall chunk takes 1.6 and 1.3, so that bricks are used
// only where latency decides (choose_brick in relax.cpp).  The arithmetic of a node is that of stage.hip
// (stage_math.h).
#include "brick.h"
#include "stage_math.h"

namespace relax {
namespace {

constexpr int NPW = (BRICK_WINDOW + BRICK_THREADS - 1) / BRICK_THREADS;  // window points per thread
constexpr int NPF = 1 + (BRICK_SHELL + BRICK_THREADS - 1) / BRICK_THREADS;  // field points per thread

template <int S, bool MIXED, bool NNN, bool DIAG = false, bool REC = false>
__global__ __launch_bounds__(BRICK_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void brick_kernel(SweepArgs a) {
  using St = Stage<S, MIXED, NNN>;
  using T = typename St::T;
  constexpr bool STAGE1 = St::STAGE1, LAST = St::LAST, LEAN = St::LEAN, WV = St::WV, CX = St::CX, CV = St::CV;
  constexpr bool PS = St::PS;
  constexpr int NPK = St::NPK, NPKA = St::NPKA, NPS = St::NPS;
  static_assert(!DIAG || (S == 1 && !MIXED), "the diagnostics sweep is the FP64 stage-1 sweep");

  // Scalars first, in one go: each that is fetched behind a branch on another costs its latency again
  // (six such fetches stood before the first load; with the index arithmetic cut to a third, us per step
  // 16^3 46.8 -> 38.5, 32^3 periodic 65.6 -> 47.4, 80^3 periodic 149 -> 135).
  const Control* ctl = a.ctl;
  int status = 0, need_k1 = 1, cur = a.diag_buf, record = 0;
  int accepted = 0, target = 1;
  long long steps_total = 0;
  double dt = 0.0;
  if (!DIAG) {
    status = ctl->status;
    cur = ctl->cur;
    accepted = ctl->accepted;
    target = ctl->target;
    dt = ctl->dt;
    if constexpr (STAGE1) {
      need_k1 = ctl->need_k1;
      record = ctl->record;
      steps_total = ctl->steps_total;
    }
  }
  const double gamma = ctl->gamma;
  const double tau_B2 = ctl->tau_B2;

  const Geometry& g = a.g;
  const long long N = g.N;
  const Brick br(g);
  const int sx = br.sx, sxy = br.sxy, fx = br.fx, fxy = br.fxy;
  const BrickOrigin at0(br, g);
  const int tid = threadIdx.x;

  __shared__ double ys[3][BRICK_WINDOW];
  __shared__ T bs[3][BRICK_FIELD];
  __shared__ double red[BRICK_THREADS / 64][NPART];

  // ---- the window and B0 first; a wave skips the points past the brick's
  double wx[NPW][3];
  T wk[WV ? NPW : 1][3];
  BrickPoint wp[NPW];
  wp[0] = brick_window(br, g, min(tid, br.nwin - 1), at0);
  const double* __restrict__ xn = cur ? a.x[1] : a.x[0];
  const double* __restrict__ wbase = (S == 3) ? a.y3 : ((S == 5) ? a.y5 : xn);
  const T* __restrict__ wvec = static_cast<const T*>(S == 2 ? a.k[0] : (S == 4 ? a.d4 : a.sum[0]));
  const T* __restrict__ b0p = static_cast<const T*>(a.B0);
  if (!DIAG && (status != 0 || accepted >= target)) return;
  if (!DIAG && STAGE1 && need_k1 == 0) return;
#pragma unroll
  for (int r = 0; r < NPW; r++) {
    const int e = tid + r * BRICK_THREADS;
    if (r == 0 || e < br.nwin) {
      if (r > 0) wp[r] = brick_window(br, g, e, at0);
      const unsigned i = wp[r].index;
#pragma unroll
      for (int m = 0; m < 3; m++) wx[r][m] = at(wbase + m * N, i);
      if constexpr (WV) {
#pragma unroll
        for (int m = 0; m < 3; m++) wk[r][m] = at(wvec + m * N, i);
      }
    }
  }
  T b0r[NPF][3];
  BrickField fp[NPF];
#pragma unroll
  for (int r = 0; r < NPF; r++) {
    fp[r].slot = -1;
    if (r == 0 || tid + (r - 1) * BRICK_THREADS < br.nshell) {
      fp[r] = brick_field(br, g, r, tid, at0);
#pragma unroll
      for (int m = 0; m < 3; m++) b0r[r][m] = at(b0p + m * N, (unsigned)fp[r].index);
    }
  }
  const bool node = fp[0].node();
  const int own = fp[0].index;
  const bool face = fp[0].face();
  const double cv = (S == 2) ? dt * CK::a[1][0] : 1.0;
  bool record_ck = false;
  long long ck_slot = 0;
  if (!DIAG && STAGE1 && record) {
    const long long every = ctl->ck_every;
    if (steps_total % every == 0 && steps_total / every < a.ckpt_slots) {
      record_ck = true;
      ck_slot = steps_total / every;
    }
  }
  // ---- stage input on the brick and its 2-node halo ------------------------------------------
#pragma unroll
  for (int r = 0; r < NPW; r++) {
    const int e = tid + r * BRICK_THREADS;
    if (e < br.nwin) {
#pragma unroll
      for (int m = 0; m < 3; m++) {
        double y = wx[r][m];
        if constexpr (S == 2) {
          y = fma(cv, (double)wk[r][m], y);
        } else if constexpr (WV) {
          y = y + (double)wk[r][m];
        }
        ys[m][e] = wp[r].on() ? y + wp[r].wrap(m) * g.period[m] : 0.0;
      }
    }
  }
  // The vectors read at the node, once the window's registers are free (4 waves a SIMD need 128); the
  // octilateral walk needs them all, so there after it.
  T pk[NPKA][3], ps[NPS][3], vq[3];
  double xq[3];
  auto load_node = [&]() {
#pragma unroll
    for (int m = 0; m < 3; m++) {
#pragma unroll
      for (int j = 0; j < NPK; j++) pk[j][m] = at(static_cast<const T*>(a.k[LEAN ? (S == 3 ? 1 : 2 * j) : j]) + m * N, own);
      if constexpr (PS) ps[0][m] = at(static_cast<const T*>(S == 5 ? a.sum[0] : a.sum[1]) + m * N, own);
      if constexpr (PS && NPS == 2) ps[NPS - 1][m] = at(static_cast<const T*>(a.sum[2]) + m * N, own);
      if constexpr (CX) xq[m] = at(xn + m * N, own);
      if constexpr (CV) vq[m] = at(wvec + m * N, own);
    }
  };
  if constexpr (!NNN) load_node();
  __syncthreads();
  const bool at_face = br.at_face(g, at0.i0, at0.j0, at0.k0);
  // ---- F', det F' and B on the brick and its 1-node halo ---------------------------------------
  Sums acc;
  T Fq[3][3], Bq[3], rDq;
  double Dq;
  int kap = 1;
#pragma unroll
  for (int r = 0; r < NPF; r++) {
    if (r == 0 || fp[r].slot >= 0) {
      const int o = fp[r].window;
      double F[3][3];
      if constexpr (NNN) {
        // the one-sided rows themselves (see stage.hip)
        auto row = [&](const double* yc, int s, int end) {
          return end == 0   ? yc[o + s] - yc[o - s]
                 : end == 1 ? -3.0 * yc[o] + 4.0 * yc[o + s] - yc[o + 2 * s]
                            : 3.0 * yc[o] - 4.0 * yc[o - s] + yc[o - 2 * s];
        };
#pragma unroll
        for (int m = 0; m < 3; m++) {
          F[m][0] = row(ys[m], 1, fp[r].ends & 3);
          F[m][1] = row(ys[m], sx, (fp[r].ends >> 2) & 3);
          F[m][2] = row(ys[m], sxy, (fp[r].ends >> 4) & 3);
        }
      } else {
        face_differences(br, fp[r].ends, at_face, ys, o, F);
      }
      const double D = (NNN || MIXED) ? det3(F) : det3_fused(F);
      const double rD = fp[r].on() ? rcp_nr(D) : 0.0;
      T q0 = b0r[r][0], q1 = b0r[r][1], q2 = b0r[r][2];
      if constexpr (DIAG) {
        q0 *= a.b0_mul[0];
        q1 *= a.b0_mul[1];
        q2 *= a.b0_mul[2];
      }
      T B[3];
      pull_back(F, q0, q1, q2, rD, B);
      if (r == 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) {
#pragma unroll
          for (int c = 0; c < 3; c++) Fq[m][c] = (T)F[m][c];
          Bq[m] = B[m];
        }
        rDq = (T)rD;
        Dq = D * g.inv8h3;
        if (STAGE1 && node) {
          double zeta = 1.0;
          if (fp[0].ends & 3) zeta *= 0.5;
          if (fp[0].ends & 12) zeta *= 0.5;
          if (fp[0].ends & 48) zeta *= 0.5;
          double Bd[3];
#pragma unroll
          for (int m = 0; m < 3; m++)
            Bd[m] = (F[m][0] * (double)q0 + F[m][1] * (double)q1 + F[m][2] * (double)q2) * rD;
          acc.E += zeta * (Bd[0] * Bd[0] + Bd[1] * Bd[1] + Bd[2] * Bd[2]) * Dq;
          acc.min_det = (Dq < acc.min_det || Dq != Dq) ? Dq : acc.min_det;
          if constexpr (DIAG) {
            double ex[2][3], ey[2][3], ez[2][3];
#pragma unroll
            for (int m = 0; m < 3; m++) {
              const double c0 = ys[m][o];
              ex[0][m] = ys[m][o - 1] - c0;
              ex[1][m] = ys[m][o + 1] - c0;
              ey[0][m] = ys[m][o - sx] - c0;
              ey[1][m] = ys[m][o + sx] - c0;
              ez[0][m] = ys[m][o - sxy] - c0;
              ez[1][m] = ys[m][o + sxy] - c0;
            }
            const bool convex = is_convex(ex, ey, ez, !(fp[0].ends & 1), !(fp[0].ends & 2), !(fp[0].ends & 4), !(fp[0].ends & 8),
                                          !(fp[0].ends & 16), !(fp[0].ends & 32));
            acc.concave += convex ? 0.0 : 1.0;
            kap = convex ? 1 : -1;
          }
        }
      }
      if (fp[r].slot >= 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) bs[m][fp[r].slot] = B[m];
      }
    }
  }
  __syncthreads();

  // ---- current, force, velocity and the stage's outputs at the own node --------------------------
  if (node) {
    StageOut<S, MIXED, NNN, DIAG, REC> so;
    const int oy = fp[0].window, o = fp[0].slot;
    T u[3] = {T(0), T(0), T(0)};
    if constexpr (DIAG) {
#pragma unroll
      for (int m = 0; m < 3; m++) {
        so.p[0][m] = Bq[m];
        so.p[1][m] = 0.0;
      }
      so.p[2][0] = 0.0;
    }
    if (!face) {
      T J[3];
      if constexpr (NNN) {
        octilateral([&](int dx, int dy, int dz, int m) { return ys[m][oy + dz * sxy + dy * sx + dx]; },
                    [&](int dx, int dy, int dz, int m) { return (double)bs[m][o + dz * fxy + dy * fx + dx]; }, J);
      } else {
        T G[3][3];
#pragma unroll
        for (int m = 0; m < 3; m++) {
          G[0][m] = bs[m][o + 1] - bs[m][o - 1];
          G[1][m] = bs[m][o + fx] - bs[m][o - fx];
          G[2][m] = bs[m][o + fxy] - bs[m][o - fxy];
        }
        current(Fq, G, rDq, J);
      }
      if constexpr (DIAG) {
#pragma unroll
        for (int m = 0; m < 3; m++) so.p[1][m] = J[m];
        const double B2 = (double)Bq[0] * Bq[0] + (double)Bq[1] * Bq[1] + (double)Bq[2] * Bq[2];
        const double JB = (double)J[0] * Bq[0] + (double)J[1] * Bq[1] + (double)J[2] * Bq[2];
        so.p[2][0] = B2 > 0.0 ? JB / B2 : 0.0;
      }
      T f[3];
      force<NNN>(J, Bq, f);
      const T gm = (T)gamma;
      u[0] = gm * f[0];
      u[1] = gm * f[1];
      u[2] = gm * f[2];
      if constexpr (STAGE1) {
        const double F2 = (double)f[0] * f[0] + (double)f[1] * f[1] + (double)f[2] * f[2];
        const double B2 = (double)Bq[0] * Bq[0] + (double)Bq[1] * Bq[1] + (double)Bq[2] * Bq[2];
        acc.force(F2, B2, Dq, tau_B2);
      }
    }
    auto put = [&](auto* to, const auto (&v)[3]) {
#pragma unroll
      for (int m = 0; m < 3; m++)
        *reinterpret_cast<decltype(to)>(reinterpret_cast<char*>(to + m * N) + (unsigned)own * (unsigned)sizeof(*to)) = v[m];
    };
    if constexpr (DIAG) {
      const double sc = a.u_det_scale != 0.0 ? Dq * a.u_det_scale : 1.0;
      const double us[3] = {(double)u[0] * sc, (double)u[1] * sc, (double)u[2] * sc};
      if (a.u_out) put(a.u_out, us);
      if (a.B_out) put(a.B_out, so.p[0]);
      if (a.J_out) put(a.J_out, so.p[1]);
      if (a.alpha_out) a.alpha_out[own] = so.p[2][0];
      if (a.kappa_out) a.kappa_out[own] = kap;
    } else if constexpr (STAGE1) {
      put(static_cast<T*>(a.k[0]), u);
      if (record_ck) {
        const double xo[3] = {ys[0][oy], ys[1][oy], ys[2][oy]};
        put(a.ckpt + ck_slot * 3 * N, xo);
      }
    } else {
      double err[3];
      if constexpr (NNN) load_node();
      advance<S, MIXED, NNN, REC>(u, xq, vq, pk, ps, dt, so, err);
      if constexpr (S == 2) {
        put(static_cast<T*>(a.k[1]), so.k);
        put(a.y3, so.y);
      } else if constexpr (S == 3) {
        put(static_cast<T*>(a.k[2]), so.k);
        put(static_cast<T*>(a.d4), so.s[0]);
      } else if constexpr (S == 4) {
        put(a.y5, so.y);
#pragma unroll
        for (int i = 0; i < 3; i++) put(static_cast<T*>(a.sum[i]), so.s[i]);
      } else if constexpr (S == 5) {
        put(static_cast<T*>(a.sum[0]), so.s[0]);
        if constexpr (!LEAN) put(static_cast<T*>(a.sum[2]), so.s[2]);
      } else {
        put(a.xout[1 - cur], so.y);
#pragma unroll
        for (int m = 0; m < 3; m++) acc.error(err[m]);
      }
    }
    if constexpr (REC) {
      const double yo[3] = {ys[0][oy], ys[1][oy], ys[2][oy]};
      put(a.yrec[S == 4 ? 0 : 1], yo);
    }
  }
  if (STAGE1) store_sums<BRICK_THREADS, DIAG>(acc, red, a.part + (long long)blockIdx.x * NPART);
  if (LAST) store_lambda<BRICK_THREADS>(acc, red, a.lam_part + blockIdx.x);
}

template <bool MIXED, bool NNN>
hipError_t launch_brick_t(int s, const SweepArgs& a, hipStream_t st) {
  const dim3 grid(a.g.nblocks), block(BRICK_THREADS);
  switch (s) {
    case 1: hipLaunchKernelGGL((brick_kernel<1, MIXED, NNN>), grid, block, 0, st, a); break;
    case 2: hipLaunchKernelGGL((brick_kernel<2, MIXED, NNN>), grid, block, 0, st, a); break;
    case 3: hipLaunchKernelGGL((brick_kernel<3, MIXED, NNN>), grid, block, 0, st, a); break;
    case 4: hipLaunchKernelGGL((brick_kernel<4, MIXED, NNN>), grid, block, 0, st, a); break;
    case 5: hipLaunchKernelGGL((brick_kernel<5, MIXED, NNN>), grid, block, 0, st, a); break;
    case 6: hipLaunchKernelGGL((brick_kernel<6, MIXED, NNN>), grid, block, 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_brick(int s, bool mixed, const SweepArgs& a, hipStream_t st) {
  if (a.g.curl == CURL_NNN) return mixed ? hipErrorInvalidValue : launch_brick_t<false, true>(s, a, st);
  return mixed ? launch_brick_t<true, false>(s, a, st) : launch_brick_t<false, false>(s, a, st);
}

hipError_t launch_brick_rec(int s, const SweepArgs& a, hipStream_t st) {
  const dim3 grid(a.g.nblocks), block(BRICK_THREADS);
  if (s == 4)
    hipLaunchKernelGGL((brick_kernel<4, false, false, false, true>), grid, block, 0, st, a);
  else if (s == 6)
    hipLaunchKernelGGL((brick_kernel<6, false, false, false, true>), grid, block, 0, st, a);
  else
    return launch_brick_t<false, false>(s, a, st);
  return hipGetLastError();
}

hipError_t launch_brick_diagnostics(const SweepArgs& a, hipStream_t st) {
  const dim3 grid(a.g.nblocks), block(BRICK_THREADS);
  if (a.g.curl == CURL_NNN)
    hipLaunchKernelGGL((brick_kernel<1, false, true, true>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((brick_kernel<1, false, false, true>), grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace relax
