// stage.hip -- the fused Runge-Kutta stage sweep of the mimetic magneto-frictional step.
//
// One launch evaluates, for every node, the right-hand side u = gamma J x B of the
// Lagrangian relaxation (eq. "magneto friction") at the stage input
//     y_s = x_n + dt sum_{j<s} a_sj k_j                  (Cash-Karp RK5(4), Sec. 2.4)
// and stores what the later stages need.  Stage 1 also reduces the diagnostics of x_n (E_M
// with the face weights zeta, eq. "magnetic energy"; xi = max |J x B| / B^2; R2; min Delta);
// stage 6 writes x_{n+1} with the fifth-order weights and reduces the embedded error
// Lambda = max |x5 - x4|.
//
// Per node the operator is two radius-1 stencils joined by pointwise maps.  With the
// UNSCALED differences (the 1/(2h) factors cancel):
//   F'   = differences of y: y(n+e_a) - y(n-e_a), or the one-sided second-order rows
//          -3y0 + 4y1 - y2 / 3y0 - 4y1 + y2 on line-tied end nodes; on periodic axes the
//          neighbour carries the +-period coordinate shift (Sec. 2.5).  F' = F diag(2h).
//   B    = F' B0'' / det F'  with B0''_a = 4 h_b h_c B0_a, which equals F B0 / det F
//          (eq. "B transformation")
//   G'_a = B(n+e_a) - B(n-e_a)
//   J    = F' c' / det F',   c'_q = (F' e_b) . G'_a - (F' e_a) . G'_b,  (a, b, q) cyclic.
// The last line is the Stokes-loop current of Sec. 2.2 (eqs. "current discrete", "four
// surfaces", "current matrix equation") in closed form: on the diamond of the four
// in-plane neighbours the edge-averaged circulation is 2 h_a h_b c_q and the sum of the
// four triangle vectors is 2 h_a h_b (F e_a) x (F e_b) = 2 h_a h_b cof(F) e_q, so the
// paper's 3x3 system is (cof F)^T J = c, solved by J = F c / det F; with F = F' diag(1/2h)
// and G = G' diag(1/2h) every spacing factor cancels.
//
// Stage inputs.  Every stage input is x_n plus ONE rounded increment, y_s = x_n + d_s with
// d_s = dt sum_j a_sj k_j summed first: the stencil differentiates y_s twice, and on a fine
// grid a rounding of y_s is amplified by about 1/h^2 in u, so the inputs are rounded once from
// x_n (as the plain definition does) and never accumulated stage by stage.  A stencilled
// window holds at most two vectors (more overflow each XCD's L2 with halo lines); what a
// stage needs at its output node from its own window (x_n with k_1, d_4 or d_6) is carried in
// registers from the window load, three plane steps earlier, instead of being read again.
// FP64 with the nearest-neighbour current (LEAN; C4 = dt (a_41 k_1 + a_42 k_2)):
//   stage 1: window x_n                    -> k_1
//   stage 2: window x_n + dt a_21 k_1      -> C4, y_3 = x_n + dt (a_31 k_1 + a_32 k_2)
//   stage 3: window y_3; C4 at node        -> k_3, d_4 = C4 + dt a_43 k_3
//   stage 4: window x_n + d_4; k_1, k_3    -> y_5 = x_n + d_5 and the partial sums of k_1..k_4
//            P6 = dt sum a_6j k_j, X = dt sum b5_j k_j, E = dt sum e_j k_j - mu P6
//            (e_j = b5_j - b4_j, mu = e_5 / a_65; k_2 from the own node's d_4, which is in the window)
//   stage 5: window y_5; P6 at node        -> P6 += dt a_65 k_5 (now d_6)
//   stage 6: window x_n + d_6; X, E        -> x_{n+1} = x_n + (X + dt b5_6 k_6),
//                                             Lambda = max |E + mu d_6 + dt e_6 k_6|
// k_2, k_4, k_5 and k_6 are never stored: 768 HBM bytes per node and attempt, where storing k_2
// and adding e_5 k_5 to E in stage 5 took 864 (256^3: 2.83 -> 2.52 ms per attempt).  Against
// 80-bit arithmetic the sums themselves round more, E + mu d_6 at 2.7e-17 of dt |k| rms instead of
// 2.8e-18 and d_5 at 2.1e-16 instead of 1.6e-16 (nearly equal k_j), but the rounding of the k_j
// outweighs both: the estimate as a whole is off by 3e-17 to 1.8e-16 of dt |k| rms on five grids of 16^3
// to 33^3 nodes and every kind of face, the same within 1 % for either set.  FP32-mixed keeps k_2 and
// accumulates E in stage 5, since there mu d_6 would add its FP32 rounding to E: Lambda off by 1.1e-8
// instead of 5e-9 of dt |k| in the worst case measured.  So does the octilateral current, whose runs
// that break down amplify every rounding.  Their stages 2..6:
//   stage 2: as above                      -> k_2, y_3
//   stage 3: window y_3; k_1, k_2          -> k_3, d_4
//   stage 4: window x_n + d_4; k_1..k_3    -> y_5, P6, X, E = dt sum e_j k_j
//   stage 5: window y_5; P6, E             -> P6 (now d_6), E += dt e_5 k_5
//   stage 6: as above                      -> x_{n+1}, Lambda = max |E + dt e_6 k_6|
// HBM bytes per node and attempt: 540 FP32-mixed (the k_j, d_4 and the partial sums in FP32; x_n,
// y_3 and y_5 in FP64), 864 with the octilateral.  x_{n+1} is x_n plus an increment built from the
// k_j alone, so the step keeps full relative precision however small it is.  A retried step
// (smaller dt, same x_n and k_1) starts again at stage 2, and every stored vector is rewritten
// before it is read again.  REC (the forward replay of the reverse pass) also stores y_4 and y_6 at
// the node for the reverse sweeps.
//
// Data flow: a workgroup owns a 64 x 8 (x, y) tile and marches up a z-chunk.  Each plane
// of the stage input (tile + 2-node halo, FP64) goes into an LDS ring of four planes;
// F', det F' and B are formed on the tile + 1-node halo into an LDS ring of two B planes
// (the z difference of B at the tile node uses the node's own B of the neighbouring
// planes, kept in registers); the current, force and velocity are formed on the tile one
// plane behind.  Every global access is a buffer instruction whose masked-off lanes carry
// an offset past the record count (loads return 0, stores are dropped), so the march has
// no divergent branch around a memory instruction: each load is issued one plane step
// before its use, in the same order on every step, and waited for by exact counts.
//
// What bounds it: at 256^3 a stage moves its bytes at 5.5 to 6.0 TB/s, against 6.1 of a streaming
// kernel with the same accesses; without any global access in the march the same sweep takes a
// third of the time (0.15 of 0.44 ms, stage 3).  Small grids are bound by latency: about 1.2 us of
// dependent FP64 and LDS work per plane step, and the first planes' way from HBM before it.
#include "stage_math.h"
#include "tile.h"

namespace relax {
namespace {

// S: stage 1..6.  MIXED: the k_j, the partial sums and B0 in FP32, and the stencil past F' in
// FP32.  NNN: the octilateral current.  DIAG (stage 1, FP64): the diagnostics sweep of x[diag_buf]:
// no step gating and no k_1; with REC it writes u (optionally scaled by det F), B, J, alpha* and the
// convexity where the caller asked for them, without REC only the sums (a store instruction takes its
// time even when every lane is masked off: 128^3 60 -> 53 us).  REC in FP64 stages 4 and 6: also
// store the stage input at the node, for the reverse sweeps.  FIT: tiles of g.tw x g.th nodes instead
// of 64 x 8, for grids whose x and y extents 64 x 8 tiles would cover with many idle threads
// (choose_tile in relax.cpp); a tile node is then any of the first tw th threads.  FACES: which axes may be line-tied
// (tile.h): with x or y a field point has two points of its own for F', with z two planes.  Against the
// neighbours for all, us per step 129^3 454 -> 460, 64 x 64 x 192 (z alone) 204 -> 204; a diagnostics call of 129^3,
// which forms eight determinants a node and is bound by its vector instructions, 97 -> 102.
template <int S, bool MIXED, bool NNN, bool DIAG, bool REC, bool FIT, int FACES>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void stage_kernel(SweepArgs a) {
  using T = typename std::conditional<MIXED, float, double>::type;
  // The stage-input ring holds the planes p - 1 .. p + 1 that the field of plane p reads and the
  // plane p + 2 committed meanwhile; B is written on plane p while the current of plane p - 1
  // reads its own, so one barrier per plane step is enough.  (On a line-tied z face the field reads plane 2
  // or nz - 3 instead, which is that fourth plane: plane 2 is committed once more, with the same bits, and
  // nothing is committed over nz - 3.)  NNN: the octilateral loops (Sec. 2.3)
  // of plane p - 1 read positions and B on the planes p - 2 .. p, B of plane p included: a barrier
  // before them, five planes of stage input and three of B.
  constexpr int RYS = NNN ? 5 : 4;
  constexpr int RBS = NNN ? 3 : 2;
  auto yslot = [](int p) { return NNN ? (int)((unsigned)(p + 1024 * 5) % 5u) : (p & 3); };
  auto bslot = [](int p) { return NNN ? mod3(p) : (p & 1); };
  constexpr bool STAGE1 = (S == 1);
  constexpr bool LAST = (S == 6);
  using St = Stage<S, MIXED, NNN>;
  constexpr bool LEAN = St::LEAN, WV = St::WV, CX = St::CX, CV = St::CV, PS = St::PS;
  constexpr int NPK = St::NPK, NPKA = St::NPKA, NPS = St::NPS;
  // Plane steps between a load and its use.  Stage 1 has the registers for two sets: 256^3 270 -> 260
  // us (FP64), 250 -> 236 us (mixed), a diagnostics call on raw arrays of 256^3 387 -> 374 us, of 128^3
  // 84.4 -> 81.9 us, of 56 x 56 x 168 (chunks of 4 planes) 53.0 -> 53.5.  The other stages gain at most 1 %
  // from a second set at 256^3 and lose 2 to 5 % on grids with short chunks (an extra step and a longer
  // prologue).
  constexpr int PD = (S == 1 && !NNN) ? 2 : 1;
  constexpr int NP2 = (RY2 * RX2 + NTHREADS - 1) / NTHREADS;  // stage-input points per thread
  constexpr int NP1 = (RY1 * RX1 + NTHREADS - 1) / NTHREADS;  // field points per thread
  constexpr int NPG = (6 * (RY2 + RX2) + NTHREADS - 1) / NTHREADS;  // sums beyond faces per thread
  static_assert(!DIAG || (S == 1 && !MIXED), "the diagnostics sweep is the FP64 stage-1 sweep");
  static_assert(!REC || DIAG || (!MIXED && (S == 4 || S == 6)), "REC: FP64 stages 4 and 6");
  static_assert(!NNN || (!MIXED && FACES == FACES_Z && (DIAG || !REC)), "the octilateral current is an FP64 forward operator");
  constexpr bool YREC = REC && !DIAG;

  // Scalars first, in one go: each that is fetched behind a branch on another costs its latency again
  const Control* ctl = a.ctl;
  constexpr bool diag_only = DIAG;
  int status = 0, need_k1 = 1, cur = a.diag_buf, record = 0;
  int accepted = 0, target = 1;
  double dt = 0.0;
  if (!diag_only) {
    status = ctl->status;
    cur = ctl->cur;
    accepted = ctl->accepted;
    target = ctl->target;
    dt = ctl->dt;
    if constexpr (STAGE1) {
      need_k1 = ctl->need_k1;
      record = ctl->record;
    }
  }
  const double gamma = ctl->gamma;
  const double tau_B2 = ctl->tau_B2;
  const double cv = (S == 2) ? dt * CK::a[1][0] : 1.0;

  const Geometry& g = a.g;
  // the tile and its windows
  const int tw = FIT ? g.tw : TX, th = FIT ? g.th : TY;
  const int wx2 = tw + 4, wy2 = th + 4, wx1 = tw + 2, wy1 = th + 2, nown = tw * th;
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const long long N = g.N;
  const int bcx = g.bc[0], bcy = g.bc[1], bcz = g.bc[2];
  const double inv8h3 = g.inv8h3;
  const unsigned nxy = (unsigned)nx * (unsigned)ny;

  const int lb = logical_block(blockIdx.x, g.nblocks);
  const int tile_x = lb % g.tiles[0];
  const int tile_y = (lb / g.tiles[0]) % g.tiles[1];
  const int chunk = lb / (g.tiles[0] * g.tiles[1]);
  const int i0 = tile_x * tw, j0 = tile_y * th;
  const int z0 = chunk * g.tz;
  const int z1 = min(z0 + g.tz, nz);

  const int tid = threadIdx.x;
  const bool own = !FIT || tid < nown;
  auto div = [](int e, int d) { return FIT ? small_div(e, d) : e / d; };
  const int ty = own ? div(tid, tw) : 0, tx = own ? tid - ty * tw : 0;

  __shared__ double ys[RYS][3][RY2 * RX2];  // stage input, tile + 2-node halo, ring of planes
  __shared__ T bs[RBS][3][RY1 * RX1];       // pulled-back field, tile + 1-node halo, ring of planes
  __shared__ double red[NTHREADS / 64][NPART];

  const double* __restrict__ xn = cur ? a.x[1] : a.x[0];
  const double* __restrict__ wbase = (S == 3) ? a.y3 : ((S == 5) ? a.y5 : xn);  // the window base
  const T* __restrict__ wvec = static_cast<const T*>(S == 2 ? a.k[0] : (S == 4 ? a.d4 : a.sum[0]));
  const T* __restrict__ b0p = static_cast<const T*>(a.B0);

  // plane index of a load (line-tied z: clamped; such planes are loaded but never used)
  auto zload = [&](int pz) {
    if (FACES == FACES_NONE || bcz == BC_PERIODIC) return resolve_near(pz, nz, BC_PERIODIC).i;
    return min(max(pz, 0), nz - 1);
  };

  // ---- per-thread index tables: the (x, y) part of every address is the same on all planes.
  // Window point e < nown is the tile node of thread e (each thread loads its own node), then
  // come the two rows below and the two above the tile, then the two columns on either side.
  unsigned w2e[NP2];  // stage-input window point -> flat (x, y) index, IE off the grid
  int w2w[NP2];       // its periodic wraps: x in the low 16 bits, y in the high 16 bits (signed)
  int w2o[NP2];       // its LDS offset, -1 past the window
#pragma unroll
  for (int r = 0; r < NP2; r++) {
    const int e = tid + r * NTHREADS;
    const auto [row, col] = window_point(e, tw, th, div);
    const bool in_win = e < wy2 * wx2;
    const AxisIdx rx = axis_index(i0 + col - 2, nx, bcx);
    const AxisIdx ry = axis_index(j0 + row - 2, ny, bcy);
    w2e[r] = (in_win && rx.ok && ry.ok) ? (unsigned)(ry.i * nx + rx.i) : IE;
    w2w[r] = (ry.w << 16) + (rx.w & 0xffff);
    w2o[r] = in_win ? row * wx2 + col : -1;
  }
  // ---- loads of one plane, issued one plane step ahead of their use -------------------------
  struct Nodes {
    T b0[NP1][3];   // B0'' at the field points
    T pk[NPKA][3];  // k_j (or C4) at the output node (stages 3, 4)
    T ps[NPS][3];   // stage 5: P6 (and E, not lean); stage 6: X, E at the output node
  };
  struct Window {
    double x[NP2][3];      // window base (x_n, y_3 or y_5)
    T v[WV ? NP2 : 1][3];  // the window vector
  };
  auto load_window = [&](Window& w, int pz, bool on) {
    const long long zo = (long long)zload(pz) * nxy;
    unsigned e[NP2];
#pragma unroll
    for (int r = 0; r < NP2; r++) e[r] = on ? w2e[r] : IE;
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const auto rs = plane_rsrc(wbase + m * N + zo, nxy);
#pragma unroll
      for (int r = 0; r < NP2; r++) w.x[r][m] = bload<double>(rs, e[r]);
    }
    if constexpr (WV) {
#pragma unroll
      for (int m = 0; m < 3; m++) {
        const auto rs = plane_rsrc(wvec + m * N + zo, nxy);
#pragma unroll
        for (int r = 0; r < NP2; r++) w.v[r][m] = bload<T>(rs, e[r]);
      }
    }
  };
  // planes of B this chunk needs
  const bool perz = FACES == FACES_NONE || bcz == BC_PERIODIC;
  const int pb0 = perz ? z0 - 1 : max(z0 - 1, 0);
  const int pb1 = perz ? z1 : min(z1, nz - 1);
  const int pw1 = perz ? pb1 + 1 : min(pb1 + 1, nz - 1);  // last plane of the stage input

  // The first three planes go out here, so that the rest of the tables is built while they are under
  // way; with the scalars above and tables without divisions, us per step: 64 x 64 x 192 176 -> 168,
  // 96^3 206 -> 197, 129^3 450 -> 438, 256^3 2404 -> 2393.
  if (!diag_only && (status != 0 || accepted >= target)) return;
  if (!diag_only && STAGE1 && need_k1 == 0) return;
  const bool low = !perz && pb0 == 0;  // the plane below holds the sums of the face
  const int lo = low ? 0 : pb0 - 1;
  Window w0, w1, w2;
  load_window(w0, lo, true);
  load_window(w1, lo + 1, true);
  load_window(w2, lo + 2, true);
  __builtin_amdgcn_sched_barrier(0);

  // field point e: e < nown is the tile node of thread e; the rest is the halo ring
  unsigned f1e[NP1];  // flat (x, y) index, IE off the grid
  int f1o[NP1];       // offset in the B window, -1 past it
  int f1y[NP1];       // offset in the stage-input window
  int f1k[NP1];       // line-tied ends it lies on: 1, 2 along x, 4, 8 along y
  int f1dx[NP1], f1dy[NP1];  // offsets of the two points whose difference is F' along x, along y: plus | minus << 16
#pragma unroll
  for (int r = 0; r < NP1; r++) {
    const int e = tid + r * NTHREADS;
    const TilePoint pt = field_point(e, tw, th, div);
    const int r1 = pt.row, c1 = pt.col;
    const bool in_win = e < wy1 * wx1;
    const AxisIdx rx = axis_index(i0 + c1 - 1, nx, bcx), ry = axis_index(j0 + r1 - 1, ny, bcy);
    f1e[r] = (in_win && rx.ok && ry.ok) ? (unsigned)(ry.i * nx + rx.i) : IE;
    f1o[r] = in_win ? r1 * wx1 + c1 : -1;
    f1y[r] = field_offset(pt, in_win, tw);
    f1k[r] = 0;
    if (bcx == BC_LINE_TIED) f1k[r] |= rx.i == 0 ? 1 : (rx.i == nx - 1 ? 2 : 0);
    if (bcy == BC_LINE_TIED) f1k[r] |= ry.i == 0 ? 4 : (ry.i == ny - 1 ? 8 : 0);
    f1dx[r] = difference_points(f1y[r], 1, f1k[r] & 3);
    f1dy[r] = difference_points(f1y[r], wx2, f1k[r] >> 2);
  }
  // NNN: points off the grid take no field (B stays 0 there, and no node off a face reads it), nor does a
  // wave without a node: narrow line-tied grids are mostly such points (us per step, 4 x 4 x 65536 11173 ->
  // 9837, 1024 x 4 x 1024 2887 -> 2782, 66 x 66 x 500 1110 -> 1078, 160^3 as before)
  int pb1_own = pb1;
  if constexpr (NNN) {
#pragma unroll
    for (int r = 0; r < NP1; r++) {
      if (f1e[r] == IE && f1o[r] >= 0) {
#pragma unroll
        for (int i = 0; i < RBS; i++)
#pragma unroll
          for (int m = 0; m < 3; m++) bs[i][m][f1o[r]] = T(0);
      }
    }
    if (!__any(f1e[0] != IE)) pb1_own = -2;
  }
  // Just beyond a line-tied face stands the sum 4 y(1) - 3 y(0) of the face node's one-sided row, which is its
  // difference from y(2): a face node differs from the others by the two points it takes, not by its path.
  // Beyond faces across x and y a thread fills one component of one row of a plane; beyond faces across z
  // see commit_sum_plane.
  const int NGC = 3 * wy2, NGR = 3 * wx2;  // sums of one column, of one row
  int gh_o[NPG], gh_s[NPG];  // offset in the plane's three components (-1: none), step into the grid
#pragma unroll
  for (int r = 0; r < NPG; r++) {
    gh_o[r] = -1;
    gh_s[r] = 0;
    const int t = tid + r * NTHREADS;
    if (t < 2 * NGC) {
      const int side = t >= NGC, t1 = t - side * NGC, m = div(t1, wy2), row = t1 - m * wy2;
      const int col = side == 0 ? 1 - i0 : nx - i0 + 2;
      if (bcx == BC_LINE_TIED && col >= 0 && col < wx2) {
        gh_o[r] = m * (RY2 * RX2) + row * wx2 + col;
        gh_s[r] = side == 0 ? 1 : -1;
      }
    } else if (t < 2 * NGC + 2 * NGR) {
      const int t0 = t - 2 * NGC, side = t0 >= NGR, t1 = t0 - side * NGR, m = div(t1, wx2), col = t1 - m * wx2;
      const int row = side == 0 ? 1 - j0 : ny - j0 + 2;
      if (bcy == BC_LINE_TIED && row >= 0 && row < wy2) {
        gh_o[r] = m * (RY2 * RX2) + row * wx2 + col;
        gh_s[r] = side == 0 ? wx2 : -wx2;
      }
    }
  }

  // tile node owned by this thread
  const int gi_t = i0 + tx, gj_t = j0 + ty;
  const bool tile_ok = own && (gi_t < nx) && (gj_t < ny);
  const unsigned out_e = tile_ok ? (unsigned)(gj_t * nx + gi_t) : IE;
  const bool face_x = bcx == BC_LINE_TIED && (gi_t == 0 || gi_t == nx - 1);
  const bool face_y = bcy == BC_LINE_TIED && (gj_t == 0 || gj_t == ny - 1);

  bool record_ck = false;
  long long ck_slot = 0;
  if (!diag_only && STAGE1 && record) {
    const long long st = ctl->steps_total, every = ctl->ck_every;
    if (st % every == 0 && st / every < a.ckpt_slots) {
      record_ck = true;
      ck_slot = st / every;
    }
  }
  // y = base + cv v, rounded once, plus the periodic shift of a wrapped neighbour
  auto window_value = [&](const Window& w, int r, double shz, double v[3]) {
#pragma unroll
    for (int m = 0; m < 3; m++) {
      double y = w.x[r][m];
      if constexpr (S == 2) {
        y = fma(cv, (double)w.v[r][m], y);
      } else if constexpr (WV) {
        y = y + (double)w.v[r][m];
      }
      v[m] = y;
    }
    v[0] += (double)(short)(w2w[r] & 0xffff) * g.period[0];
    v[1] += (double)(w2w[r] >> 16) * g.period[1];
    v[2] += shz;
  };
  auto commit_window = [&](const Window& w, int pz) {
    const double shz = resolve_near(pz, nz, bcz).w * g.period[2];
    const int slot = yslot(pz);
#pragma unroll
    for (int r = 0; r < NP2; r++) {
      double v[3];
      window_value(w, r, shz, v);
      if (w2o[r] >= 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) ys[slot][m][w2o[r]] = (w2e[r] != IE) ? v[m] : 0.0;
      }
    }
  };
  // the sums of a line-tied z face, in the plane beyond it, from the face's plane pa and the next, pb: each
  // thread reads back the points it committed itself.  NNN: only the diagnostics' edge vectors read them,
  // whose trihedra there are not formed
  auto commit_sum_plane = [&](int pz, int pa, int pb) {
    const int slot = yslot(pz), sa = yslot(pa), sb = yslot(pb);
#pragma unroll
    for (int r = 0; r < NP2; r++) {
      if (w2o[r] >= 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) ys[slot][m][w2o[r]] = face_sum(ys[sa][m][w2o[r]], ys[sb][m][w2o[r]]);
      }
    }
  };
  // no field point of the tile lies on a line-tied face across x or y
  const bool inner_xy = (bcx == BC_PERIODIC || (i0 > 0 && i0 + tw + 1 < nx)) &&
                        (bcy == BC_PERIODIC || (j0 > 0 && j0 + th + 1 < ny));
  // NNN: the one-sided rows themselves.  (The octilateral runs that break down amplify the rounding
  // of the face rows, so these keep the order of operations they have always had.)
  auto jacobian_rows = [&](int o, int ends, int p, double F[3][3]) {
    const int sp = yslot(p);
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const double* yc = ys[sp][m];
      if (!(ends & 3))
        F[m][0] = yc[o + 1] - yc[o - 1];
      else if (ends & 1)
        F[m][0] = -3.0 * yc[o] + 4.0 * yc[o + 1] - yc[o + 2];
      else
        F[m][0] = 3.0 * yc[o] - 4.0 * yc[o - 1] + yc[o - 2];
      if (!(ends & 12))
        F[m][1] = yc[o + wx2] - yc[o - wx2];
      else if (ends & 4)
        F[m][1] = -3.0 * yc[o] + 4.0 * yc[o + wx2] - yc[o + 2 * wx2];
      else
        F[m][1] = 3.0 * yc[o] - 4.0 * yc[o - wx2] + yc[o - 2 * wx2];
    }
    if (bcz == BC_PERIODIC || (p > 0 && p < nz - 1)) {
      const int sa = yslot(p + 1), sb = yslot(p - 1);
#pragma unroll
      for (int m = 0; m < 3; m++) F[m][2] = ys[sa][m][o] - ys[sb][m][o];
    } else if (p == 0) {
#pragma unroll
      for (int m = 0; m < 3; m++) F[m][2] = -3.0 * ys[yslot(0)][m][o] + 4.0 * ys[yslot(1)][m][o] - ys[yslot(2)][m][o];
    } else {
      const int s0 = yslot(p), s1 = yslot(p - 1), s2 = yslot(p - 2);
#pragma unroll
      for (int m = 0; m < 3; m++) F[m][2] = 3.0 * ys[s0][m][o] - 4.0 * ys[s1][m][o] + ys[s2][m][o];
    }
  };
  auto fill_sums = [&](int pz) {
    if constexpr (FACES != FACES_XY) return;
#pragma unroll
    for (int r = 0; r < NPG; r++) {
      if (gh_o[r] >= 0) {
        double* y = &ys[yslot(pz)][0][gh_o[r]];
        *y = face_sum(y[gh_s[r]], y[2 * gh_s[r]]);
      }
    }
  };
  // own-node values (window point 0) of the planes p - 1, p, p + 1, oldest first
  double cx[CX ? 3 : 1][3] = {};
  T cvv[CV ? 3 : 1][3] = {};
  auto carry = [&](const Window& w) {
#pragma unroll
    for (int m = 0; m < 3; m++) {
      if constexpr (CX) {
        cx[0][m] = cx[1][m];
        cx[1][m] = cx[2][m];
        cx[2][m] = w.x[0][m];
        pin(cx[2][m]);
      }
      if constexpr (CV) {
        cvv[0][m] = cvv[1][m];
        cvv[1][m] = cvv[2][m];
        cvv[2][m] = w.v[0][m];
        pin(cvv[2][m]);
      }
    }
  };
  auto load_b0 = [&](Nodes& nd, int pz) {
    const long long zo = (long long)zload(pz) * nxy;
#pragma unroll
    for (int m = 0; m < 3; m++) {
      const auto rs = plane_rsrc(b0p + m * N + zo, nxy);
#pragma unroll
      for (int r = 0; r < NP1; r++) nd.b0[r][m] = bload<T>(rs, f1e[r]);
    }
  };
  auto load_point = [&](Nodes& nd, int pz) {
    const long long zo = (long long)zload(pz) * nxy;
    const unsigned eo = (pz >= z0 && pz < z1) ? out_e : IE;
    if constexpr (NPK > 0) {
#pragma unroll
      for (int j = 0; j < NPK; j++) {
        const T* kj = static_cast<const T*>(a.k[LEAN ? (S == 3 ? 1 : 2 * j) : j]);
#pragma unroll
        for (int m = 0; m < 3; m++) nd.pk[j][m] = bload<T, CPOL_STREAM>(plane_rsrc(kj + m * N + zo, nxy), eo);
      }
    }
    if constexpr (PS) {
      const T* s0 = static_cast<const T*>(S == 5 ? a.sum[0] : a.sum[1]);
      const T* s1 = static_cast<const T*>(a.sum[2]);
#pragma unroll
      for (int m = 0; m < 3; m++) nd.ps[0][m] = bload<T, CPOL_STREAM>(plane_rsrc(s0 + m * N + zo, nxy), eo);
#pragma unroll
      for (int m = 0; m < 3 && NPS == 2; m++) nd.ps[NPS - 1][m] = bload<T, CPOL_STREAM>(plane_rsrc(s1 + m * N + zo, nxy), eo);
    }
  };

  Sums acc;

  // ---- stores of one output plane (every lane issues them; masked-off lanes are dropped) ----
  using Outputs = StageOut<S, MIXED, NNN, DIAG, REC>;
  auto store_plane = [&](const Outputs& so, int qz, bool on, int kap = 1) {
    const long long zo = (long long)zload(qz) * nxy;
    const unsigned eo = on ? out_e : IE;
    if constexpr (DIAG && !REC) {
      (void)eo;
    } else if constexpr (DIAG) {
      // each output goes to the caller's array, or (masked) to x[diag_buf], never written
      double* fb = const_cast<double*>(a.x[cur]);
      double* du = a.u_out ? a.u_out : fb;
      double* dB = a.B_out ? a.B_out : fb;
      double* dJ = a.J_out ? a.J_out : fb;
      const unsigned eu = (on && a.u_out) ? out_e : IE, eB = (on && a.B_out) ? out_e : IE;
      const unsigned eJ = (on && a.J_out) ? out_e : IE;
      double* dA = a.alpha_out ? a.alpha_out : fb;
      int* dK = a.kappa_out ? a.kappa_out : reinterpret_cast<int*>(fb);
      const unsigned eA = (on && a.alpha_out) ? out_e : IE, eK = (on && a.kappa_out) ? out_e : IE;
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(du + m * N + zo, nxy), eu, (double)so.k[m]);
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(dB + m * N + zo, nxy), eB, so.p[0][m]);
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(dJ + m * N + zo, nxy), eJ, so.p[1][m]);
      bstore<double>(plane_rsrc(dA + zo, nxy), eA, so.p[2][0]);
      bstore<int>(plane_rsrc(dK + zo, nxy), eK, kap);
    } else if constexpr (STAGE1) {
      const unsigned ec = (on && record_ck) ? out_e : IE;
      T* dk = static_cast<T*>(a.k[0]);
      double* dc = record_ck ? a.ckpt + ck_slot * 3 * N : a.xout[0];
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<T>(plane_rsrc(dk + m * N + zo, nxy), eo, so.k[m]);
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(dc + m * N + zo, nxy), ec, so.y[m]);
    } else if constexpr (S == 2) {
      T* dk = static_cast<T*>(a.k[1]);
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<T>(plane_rsrc(dk + m * N + zo, nxy), eo, so.k[m]);
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(a.y3 + m * N + zo, nxy), eo, so.y[m]);
    } else if constexpr (S == 3) {
      T* dk = static_cast<T*>(a.k[2]);
      T* dd = static_cast<T*>(a.d4);
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<T>(plane_rsrc(dk + m * N + zo, nxy), eo, so.k[m]);
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<T>(plane_rsrc(dd + m * N + zo, nxy), eo, so.s[0][m]);
    } else if constexpr (S == 4) {
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(a.y5 + m * N + zo, nxy), eo, so.y[m]);
#pragma unroll
      for (int i = 0; i < 3; i++) {
        T* ds = static_cast<T*>(a.sum[i]);
#pragma unroll
        for (int m = 0; m < 3; m++) bstore<T>(plane_rsrc(ds + m * N + zo, nxy), eo, so.s[i][m]);
      }
    } else if constexpr (S == 5) {
#pragma unroll
      for (int i = 0; i < (LEAN ? 1 : 3); i += 2) {
        T* ds = static_cast<T*>(a.sum[i]);
#pragma unroll
        for (int m = 0; m < 3; m++) bstore<T>(plane_rsrc(ds + m * N + zo, nxy), eo, so.s[i][m]);
      }
    } else {
      double* xo = a.xout[1 - cur];
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(xo + m * N + zo, nxy), eo, so.y[m]);
    }
    if constexpr (YREC) {
      double* dy = a.yrec[S == 4 ? 0 : 1];
#pragma unroll
      for (int m = 0; m < 3; m++) bstore<double>(plane_rsrc(dy + m * N + zo, nxy), eo, so.yc[m]);
    }
  };

  Window win[PD];
  Nodes nodes[PD];
  auto commit_next = [&](const Window& win, int p) {
    // past the chunk's last plane: zeros that nothing reads; beyond a face the sums, and then nothing, since
    // plane nz - 3 is still wanted for the row
    if (perz || p + 2 < nz)
      commit_window(win, p + 2);
    else if ((!NNN || DIAG) && p + 2 == nz)
      commit_sum_plane(nz, nz - 1, nz - 2);
    carry(win);
  };

  // ---- prologue: the stage input on the planes pb0 - 1 .. pb0 + 1
  {
    commit_window(w0, lo);
    commit_window(w1, lo + 1);
    commit_window(w2, lo + 2);
    if (low) {  // plane 2 stays in the ring; the first plane step commits it again, with the same bits
      if constexpr (!NNN || DIAG) commit_sum_plane(-1, 0, 1);
      carry(w0);
      carry(w0);
      carry(w1);
    } else {
      carry(w0);
      carry(w1);
      carry(w2);
    }
  }
  __syncthreads();
  fill_sums(pb0);
  // leave the same loads and (dropped) stores in flight, in the same order, as a plane step
#pragma unroll
  for (int d = 0; d < PD; d++) {
    if constexpr (!NNN) load_window(win[d], pb0 + d + 2, pb0 + d + 2 <= pw1);
    load_b0(nodes[d], min(pb0 + d, pb1));
    load_point(nodes[d], pb0 + d - 1);
    store_plane(Outputs{}, pb0 + d - 1, false);
    if constexpr (NNN) load_window(win[d], pb0 + d + 2, pb0 + d + 2 <= pw1);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();

  // own-node values carried between plane steps: B at q - 1 and q; at q: F', 1 / det F', det F
  T Bqm[3] = {T(0), T(0), T(0)}, Bq[3] = {T(0), T(0), T(0)};
  T Fq[3][3] = {};
  T rDq = T(0);
  double Dq = 0.0;
  int kap_q = 1;  // DIAG: convexity

  auto step = [&](int p, Nodes& nd, Window& win) {
    const int q = p - 1;
    const bool qout = (q >= z0 && q < z1);
    fill_sums(p + 1);
    // own-node values of plane q
    double xq[3] = {0.0, 0.0, 0.0};
    T vq[3] = {T(0), T(0), T(0)};
#pragma unroll
    for (int m = 0; m < 3; m++) {
      if constexpr (CX) xq[m] = cx[0][m];
      if constexpr (CV) vq[m] = cvv[0][m];
    }
    // 0. commit the plane the next field needs and load the one after it.  First, so that the window
    // loads go out while the field is computed, and not in one burst with the stores at the end of the
    // step (256^3, stage 3: 375 -> 354 us, stage 5: 312 -> 285)
    if constexpr (!NNN) {
      commit_next(win, p);
      load_window(win, p + PD + 2, p + PD + 2 <= pw1);
    }
    // 1. F', det F' and B of field point R of plane p; off the grid B = 0
    T Bp[3], Fp[3][3], rDp;
    double Dp;
    int kap_p = 1;
    const bool central = inner_xy && (perz || (p > 0 && p < nz - 1));
    // the planes whose difference is F' along z (line-tied faces: the sum and plane 2 or nz - 3)
    const bool low_face = !perz && p == 0, high_face = !perz && p == nz - 1;
    const int sp = yslot(low_face ? -1 : (high_face ? p - 2 : p + 1));
    const int sm = yslot(low_face ? 2 : (high_face ? p + 1 : p - 1));
    auto field = [&](auto point) {
      constexpr int R = decltype(point)::value;
      const int sb = bslot(p);
      const bool ok = (f1e[R] != IE);
      T B[3];
      const int o = f1y[R];
      const int sc = yslot(p), sl = yslot(p - 1), sh = yslot(p + 1);
      double F[3][3];
      if (NNN && !central) {
        jacobian_rows(o, f1k[R], p, F);
      } else {
#pragma unroll
        for (int m = 0; m < 3; m++) {
          if constexpr (FACES == FACES_XY) {
            F[m][0] = ys[sc][m][f1dx[R] & 0xffff] - ys[sc][m][f1dx[R] >> 16];
            F[m][1] = ys[sc][m][f1dy[R] & 0xffff] - ys[sc][m][f1dy[R] >> 16];
          } else {
            F[m][0] = ys[sc][m][o + 1] - ys[sc][m][o - 1];
            F[m][1] = ys[sc][m][o + wx2] - ys[sc][m][o - wx2];
          }
          F[m][2] = ys[NNN ? sh : sp][m][o] - ys[NNN ? sl : sm][m][o];
        }
      }
      const double D = (NNN || MIXED) ? det3(F) : det3_fused(F);
      const double rD = ok ? rcp_nr(D) : 0.0;
      T q0 = nd.b0[R][0], q1 = nd.b0[R][1], q2 = nd.b0[R][2];
      if constexpr (DIAG) {
        q0 *= a.b0_mul[0];
        q1 *= a.b0_mul[1];
        q2 *= a.b0_mul[2];
      }
      pull_back(F, q0, q1, q2, rD, B);
      if constexpr (R == 0) {  // this thread's own tile node
#pragma unroll
        for (int m = 0; m < 3; m++) {
#pragma unroll
          for (int c = 0; c < 3; c++) Fp[m][c] = (T)F[m][c];
          Bp[m] = B[m];
        }
        rDp = (T)rD;
        Dp = D * inv8h3;
        if (STAGE1 && p >= z0 && p < z1 && tile_ok) {
          // energy in FP64 from the FP64 Jacobian and B0'', weights zeta on line-tied faces
          double zeta = 1.0;
          if (face_x) zeta *= 0.5;
          if (face_y) zeta *= 0.5;
          if (bcz == BC_LINE_TIED && (p == 0 || p == nz - 1)) zeta *= 0.5;
          double Bd[3];
#pragma unroll
          for (int m = 0; m < 3; m++)
            Bd[m] = (F[m][0] * (double)q0 + F[m][1] * (double)q1 + F[m][2] * (double)q2) * rD;
          acc.E += zeta * (Bd[0] * Bd[0] + Bd[1] * Bd[1] + Bd[2] * Bd[2]) * Dp;
          acc.min_det = (Dp < acc.min_det || Dp != Dp) ? Dp : acc.min_det;
          if constexpr (DIAG) {
            const bool lox = bcx == BC_PERIODIC || gi_t > 0, hix = bcx == BC_PERIODIC || gi_t < nx - 1;
            const bool loy = bcy == BC_PERIODIC || gj_t > 0, hiy = bcy == BC_PERIODIC || gj_t < ny - 1;
            const bool loz = bcz == BC_PERIODIC || p > 0, hiz = bcz == BC_PERIODIC || p < nz - 1;
            double ex[2][3], ey[2][3], ez[2][3];  // [0]: toward -, [1]: toward +
#pragma unroll
            for (int m = 0; m < 3; m++) {
              const double c0 = ys[sc][m][o];
              ex[0][m] = ys[sc][m][o - 1] - c0;
              ex[1][m] = ys[sc][m][o + 1] - c0;
              ey[0][m] = ys[sc][m][o - wx2] - c0;
              ey[1][m] = ys[sc][m][o + wx2] - c0;
              ez[0][m] = ys[sl][m][o] - c0;
              ez[1][m] = ys[sh][m][o] - c0;
            }
            const bool convex = is_convex(ex, ey, ez, lox, hix, loy, hiy, loz, hiz);
            acc.concave += convex ? 0.0 : 1.0;
            kap_p = convex ? 1 : -1;
          }
        }
      }
      if (!FIT || R > 0 || f1o[R] >= 0) {
#pragma unroll
        for (int m = 0; m < 3; m++) bs[sb][m][f1o[R]] = B[m];
      }
    };
    static_assert(NP1 == 2 && RY1 * RX1 >= NTHREADS, "one tile node and at most one halo point per thread");
    using OwnNode = std::integral_constant<int, 0>;
    using HaloPoint = std::integral_constant<int, 1>;
    if constexpr (NNN) {
      if (p <= pb1_own) field(OwnNode{});
      __builtin_amdgcn_sched_barrier(0);  // one field point at a time: bounds live temporaries
      if (p <= pb1 && f1e[1] != IE) field(HaloPoint{});
    } else {
      // the halo points first (three of the eight waves); past the chunk's last plane the field is
      // computed too and not read
      if (f1o[1] >= 0) field(HaloPoint{});
      field(OwnNode{});
    }
    load_b0(nd, min(p + PD, pb1));
    // the octilateral walk needs many registers: the window is committed before it and loaded
    // after it, so that no window value is live across it
    if constexpr (NNN) {
      __syncthreads();
      commit_next(win, p);
    }

    // 2. current, force and velocity on the tile of plane q = p - 1
    Outputs so;
    if (qout) {
      const int oy = (ty + 2) * wx2 + tx + 2;  // the tile node in the window
      if constexpr (YREC) {
#pragma unroll
        for (int m = 0; m < 3; m++) so.yc[m] = ys[yslot(q)][m][oy];
      }
      const bool face = face_x || face_y || (bcz == BC_LINE_TIED && (q == 0 || q == nz - 1));
      T u[3] = {T(0), T(0), T(0)};
      if constexpr (DIAG) {
#pragma unroll
        for (int m = 0; m < 3; m++) {
          so.p[0][m] = Bq[m];
          so.p[1][m] = 0.0;  // J: zero on line-tied faces
        }
        so.p[2][0] = 0.0;
      }
      if (!NNN || !face) {
        const int o = (ty + 1) * wx1 + (tx + 1);
        const int sq = bslot(q);
        T J[3];
        if constexpr (NNN) {
          octilateral([&](int dx, int dy, int dz, int m) { return ys[yslot(q + dz)][m][oy + dy * wx2 + dx]; },
                      [&](int dx, int dy, int dz, int m) { return (double)bs[bslot(q + dz)][m][o + dy * wx1 + dx]; }, J);
        } else {
          T G[3][3];  // G'[a][m] = B_m(n + e_a) - B_m(n - e_a)
#pragma unroll
          for (int m = 0; m < 3; m++) {
            G[0][m] = bs[sq][m][o + 1] - bs[sq][m][o - 1];
            G[1][m] = bs[sq][m][o + wx1] - bs[sq][m][o - wx1];
            G[2][m] = Bp[m] - Bqm[m];
          }
          current(Fq, G, rDq, J);
        }
        if constexpr (DIAG) {
#pragma unroll
          for (int m = 0; m < 3; m++) so.p[1][m] = face ? 0.0 : (double)J[m];
          // alpha* = J.B / B^2 (Sec. 3.2.1); 0 where B vanishes
          const double B2 = (double)Bq[0] * Bq[0] + (double)Bq[1] * Bq[1] + (double)Bq[2] * Bq[2];
          const double JB = (double)J[0] * Bq[0] + (double)J[1] * Bq[1] + (double)J[2] * Bq[2];
          so.p[2][0] = (B2 > 0.0 && !face) ? JB / B2 : 0.0;
        }
        T f[3];
        force<NNN>(J, Bq, f);
        const T gm = (T)gamma;
        u[0] = face ? T(0) : gm * f[0];
        u[1] = face ? T(0) : gm * f[1];
        u[2] = face ? T(0) : gm * f[2];
        if (STAGE1 && tile_ok && !face) {
          const double F2 = (double)f[0] * f[0] + (double)f[1] * f[1] + (double)f[2] * f[2];
          const double B2 = (double)Bq[0] * Bq[0] + (double)Bq[1] * Bq[1] + (double)Bq[2] * Bq[2];
          acc.force(F2, B2, Dq, tau_B2);
        }
      }
      if constexpr (STAGE1) {
        const double sc = (diag_only && a.u_det_scale != 0.0) ? Dq * a.u_det_scale : 1.0;
#pragma unroll
        for (int m = 0; m < 3; m++) {
          so.k[m] = diag_only ? (T)((double)u[m] * sc) : u[m];
          if constexpr (!DIAG) so.y[m] = ys[yslot(q)][m][oy];
        }
      } else {
        double err[3];
        if constexpr (FACES == FACES_NONE && !MIXED && (S == 3 || S == 5)) {  // 256^3: 362 -> 352, 299 -> 283 us
          double from[1][3];
#pragma unroll
          for (int m = 0; m < 3; m++) from[0][m] = taken(S == 3 ? nd.pk[0][m] : nd.ps[0][m]);
          advance<S, MIXED, NNN, REC>(u, xq, vq, from, from, dt, so, err);
        } else {
          advance<S, MIXED, NNN, REC>(u, xq, vq, nd.pk, nd.ps, dt, so, err);
        }
        if constexpr (LAST)
#pragma unroll
          for (int m = 0; m < 3; m++) acc.error(tile_ok ? err[m] : 0.0);
      }
    }
    load_point(nd, p + PD - 1);  // output node of the plane step that uses this set next
    store_plane(so, q, qout, kap_q);

    if constexpr (NNN) load_window(win, p + PD + 2, p + PD + 2 <= pw1);
    __syncthreads();

#pragma unroll
    for (int m = 0; m < 3; m++) {
      Bqm[m] = Bq[m];
      Bq[m] = Bp[m];
#pragma unroll
      for (int c = 0; c < 3; c++) Fq[m][c] = Fp[m][c];
    }
    rDq = rDp;
    Dq = Dp;
    kap_q = kap_p;
  };
  // with two sets, the last step may be one past z1: it writes nothing
  for (int p = pb0; p <= z1; p += PD) {
    step(p, nodes[0], win[0]);
    if constexpr (PD == 2) step(p + 1, nodes[PD - 1], win[PD - 1]);
  }

  // ---- workgroup reductions -> partial records -----------------------------------------
  if (STAGE1) store_sums<NTHREADS, DIAG>(acc, red, a.part + (long long)blockIdx.x * NPART);
  if (LAST) store_lambda<NTHREADS>(acc, red, a.lam_part + blockIdx.x);
}

template <int S, bool MIXED, bool NNN, bool DIAG, bool REC, int FACES>
hipError_t launch_tiles(const SweepArgs& a, hipStream_t st) {
  const dim3 grid(a.g.nblocks), block(NTHREADS);
  if (a.g.tw == TX && a.g.th == TY)
    hipLaunchKernelGGL((stage_kernel<S, MIXED, NNN, DIAG, REC, false, FACES>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((stage_kernel<S, MIXED, NNN, DIAG, REC, true, FACES>), grid, block, 0, st, a);
  return hipGetLastError();
}
template <int S, bool MIXED, bool NNN, bool DIAG = false, bool REC = false>
hipError_t launch_march(const SweepArgs& a, hipStream_t st) {
  if constexpr (!NNN) {
    if (faces_of(a.g) == FACES_NONE) return launch_tiles<S, MIXED, NNN, DIAG, REC, FACES_NONE>(a, st);
    if (faces_of(a.g) == FACES_XY) return launch_tiles<S, MIXED, NNN, DIAG, REC, FACES_XY>(a, st);
  }
  return launch_tiles<S, MIXED, NNN, DIAG, REC, FACES_Z>(a, st);
}

template <bool MIXED, bool NNN = false>
hipError_t launch_stage_t(int s, const SweepArgs& a, hipStream_t st) {
  switch (s) {
    case 1: return launch_march<1, MIXED, NNN>(a, st);
    case 2: return launch_march<2, MIXED, NNN>(a, st);
    case 3: return launch_march<3, MIXED, NNN>(a, st);
    case 4: return launch_march<4, MIXED, NNN>(a, st);
    case 5: return launch_march<5, MIXED, NNN>(a, st);
    case 6: return launch_march<6, MIXED, NNN>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_stage(int s, bool mixed, const SweepArgs& a, hipStream_t st) {
  if (a.g.brick[0]) return launch_brick(s, mixed, a, st);
  if (a.g.curl == CURL_NNN) return mixed ? hipErrorInvalidValue : launch_stage_t<false, true>(s, a, st);
  return mixed ? launch_stage_t<true>(s, a, st) : launch_stage_t<false>(s, a, st);
}

// the forward replay of the reverse pass (FP64): stages 4 and 6 also store their input
hipError_t launch_stage_rec(int s, const SweepArgs& a, hipStream_t st) {
  if (a.g.curl == CURL_NNN) return hipErrorInvalidValue;
  if (a.g.brick[0]) return launch_brick_rec(s, a, st);
  if (s == 4) return launch_march<4, false, false, false, true>(a, st);
  if (s == 6) return launch_march<6, false, false, false, true>(a, st);
  return launch_stage_t<false>(s, a, st);
}

hipError_t launch_diagnostics(const SweepArgs& a, hipStream_t st) {
  if (a.g.brick[0]) return launch_brick_diagnostics(a, st);
  const bool fields = a.u_out || a.B_out || a.J_out || a.alpha_out || a.kappa_out;
  if (a.g.curl == CURL_NNN)
    return fields ? launch_march<1, false, true, true, true>(a, st) : launch_march<1, false, true, true>(a, st);
  return fields ? launch_march<1, false, false, true, true>(a, st) : launch_march<1, false, false, true>(a, st);
}

}  // namespace relax
