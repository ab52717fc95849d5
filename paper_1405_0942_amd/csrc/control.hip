// control.hip -- device-side step control and the small set-up / reduction kernels.
//
// The control kernel closes one Cash-Karp attempt without a host round trip: it reduces
// the per-workgroup partials of the stage sweeps in a fixed order (deterministic), checks
// for breakdown, and applies the step-size rule of Sec. 2.4 (eq. "time stepping"):
//     dt' = dt |Lambda_0 / Lambda|^{0.2}
//     Lambda >  Lambda_0       -> reject, retry from x_n with dt'
//     Lambda <  Lambda_0 / 2   -> accept, continue with dt'
//     otherwise                -> accept, keep dt
// (Lambda == 0 grows the step 5x.)  On acceptance it records the step's diagnostics in
// the device ring and swaps the position buffers.
#include "sweep_common.h"

namespace relax {
namespace {

constexpr int CT = 256;  // workgroup size of the set-up reductions

// status codes (the values of include/relax.h)
constexpr int E_FOLD = -3, E_DT = -4, E_NAN = -5;

// The reduction of the workgroups' records: two waves per quantity, each lane a share of the records in a
// fixed order, then the lanes by DPP.  Quantity 5 of a record is `sixth` with stride `stride6`: Lambda of
// stage 6, or the concave count of a diagnostics sweep.  The loads of all quantities go out together and
// wait for nothing else, which is what the time of these kernels is made of: 64 records 4.4 -> 3.0 us, 256
// records 6.3 -> 5.0, against LDS trees of six arrays after the control block's fields one by one.
constexpr int RT = 768;
template <bool LAMBDA>
__device__ __forceinline__ void reduce_records(const double* __restrict__ part, const double* __restrict__ sixth,
                                               int stride6, int nblocks, double s[12]) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = wave % 6, half = wave / 6;
  const double* p = q == 5 ? sixth : part + q;
  const int stride = q == 5 ? stride6 : NPART;
  double sum = 0.0, X = 0.0, M = INFINITY;
#pragma unroll 4
  for (int b = half * 64 + lane; b < nblocks; b += 128) {
    const double v = p[(long long)b * stride];
    sum += v;
    X = max_nan(X, v);
    M = min_nan(M, v);
  }
  double v;
  if (q == 2 || (LAMBDA && q == 5))
    v = wave_max(X);
  else if (q == 3)
    v = wave_min(M);
  else
    v = wave_sum(sum);
  if (lane == 63) s[wave] = v;
}

__global__ __launch_bounds__(RT) void control_kernel(Control* ctl, const double* __restrict__ part,
                                                     const double* __restrict__ lam_part, int nblocks,
                                                     double* __restrict__ ring, double* __restrict__ dt_record) {
  Control c = *ctl;
  __shared__ double s[12];
  reduce_records<true>(part, lam_part, 1, nblocks, s);
  if (c.status != 0 || c.accepted >= c.target) return;
  __syncthreads();
  if (threadIdx.x != 0) return;

  if (c.need_k1 != 0) {  // x_n is new: stage 1 has left its diagnostics
    ctl->E = c.E = 0.5 * (s[0] + s[6]) * c.dV;
    ctl->R2 = c.R2 = 0.5 * (s[1] + s[7]) * c.dV;
    ctl->xi = c.xi = max_nan(s[2], s[8]);
    ctl->min_det = c.min_det = min_nan(s[3], s[9]);
    ctl->nulls = s[4] + s[10];
    ctl->need_k1 = 0;
    if (c.min_det != c.min_det) {
      ctl->status = E_NAN;
      return;
    }
    if (!(c.min_det > 0.0)) {
      ctl->status = E_FOLD;
      return;
    }
    if (!isfinite(c.E) || !isfinite(c.R2)) {
      ctl->status = E_NAN;
      return;
    }
  }
  const double lam = max_nan(s[5], s[11]);
  ctl->lambda = lam;
  if (lam != lam || isinf(lam)) {
    ctl->status = E_NAN;
    return;
  }
  const double dt = c.dt;
  double dt_next = dt;
  bool accept = true;
  if (c.adaptive) {
    const double dtp = (lam > 0.0) ? c.safety * dt * pow(fabs(c.tol / lam), 0.2) : 5.0 * dt;
    if (lam > c.tol) {
      accept = false;
      dt_next = dtp;
    } else {
      dt_next = (lam < 0.5 * c.tol) ? dtp : dt;
    }
  }
  if (!accept) {
    ctl->rejects = c.rejects + 1;
    ctl->dt = dt_next;
    if (dt_next < c.dt_min) ctl->status = E_DT;
    return;
  }
  double* e = ring + (long long)c.accepted * 8;
  e[0] = c.t;
  e[1] = dt;
  e[2] = c.E;
  e[3] = c.xi;
  e[4] = c.R2;
  e[5] = lam;
  e[6] = c.min_det;
  e[7] = (double)c.rejects;
  if (c.record && dt_record && c.steps_total < c.record_cap) dt_record[c.steps_total] = dt;
  ctl->t = c.t + dt;
  ctl->dt = dt_next;
  ctl->cur = 1 - c.cur;
  ctl->accepted = c.accepted + 1;
  ctl->steps_total = c.steps_total + 1;
  ctl->rejects = 0;
  ctl->need_k1 = 1;
}

// final reduction of a diagnostics sweep: out = {sum E, sum R2, max xi, min det, nulls, concave cells}
__global__ __launch_bounds__(RT) void diag_finish_kernel(const double* __restrict__ part, int nblocks, double dV,
                                                         double* __restrict__ out) {
  __shared__ double s[12];
  reduce_records<false>(part, part + 5, NPART, nblocks, s);
  __syncthreads();
  const int q = threadIdx.x;
  if (q < 6) {
    const double v = q == 2 ? max_nan(s[2], s[8]) : (q == 3 ? min_nan(s[3], s[9]) : s[q] + s[q + 6]);
    out[q] = q < 2 ? 0.5 * v * dV : v;
  }
}

__global__ void begin_chunk_kernel(Control* ctl, int target) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    ctl->accepted = 0;
    ctl->target = target;
  }
}

__global__ void to_float_kernel(const double* __restrict__ s, float* __restrict__ d, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    d[i] = (float)s[i];
}

// component-wise scaling of a [3][N] field in place
__global__ void prescale_kernel(double* __restrict__ v, long long N, double s0, double s1, double s2) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
    v[i] *= s0;
    v[i + N] *= s1;
    v[i + 2 * N] *= s2;
  }
}

// max over nodes of |v|^2 of a [3][N] field, in two passes (used once at set-up): each
// workgroup reduces a grid-stride share into part[blockIdx.x], then one workgroup reduces
// the partials (a max, so the result does not depend on the order)
__global__ __launch_bounds__(CT) void max_norm2_part_kernel(const double* __restrict__ v, long long N,
                                                             double* __restrict__ part) {
  __shared__ double s[CT];
  double m = 0.0;
  for (long long i = (long long)blockIdx.x * CT + threadIdx.x; i < N; i += (long long)gridDim.x * CT) {
    const double a = v[i], b = v[i + N], c = v[i + 2 * N];
    m = max_nan(m, a * a + b * b + c * c);
  }
  s[threadIdx.x] = m;
  __syncthreads();
  for (int k = CT / 2; k > 0; k >>= 1) {
    if (threadIdx.x < k) s[threadIdx.x] = max_nan(s[threadIdx.x], s[threadIdx.x + k]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// ... and, with a control block, what the diagnostics sweep of a call without a context reads from it
__global__ __launch_bounds__(CT) void max_reduce_kernel(const double* __restrict__ part, int n,
                                                        double* __restrict__ out, Control* ctl, double gamma,
                                                        double xi_null_tau) {
  __shared__ double s[CT];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += CT) m = max_nan(m, part[i]);
  s[threadIdx.x] = m;
  __syncthreads();
  for (int k = CT / 2; k > 0; k >>= 1) {
    if (threadIdx.x < k) s[threadIdx.x] = max_nan(s[threadIdx.x], s[threadIdx.x + k]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *out = s[0];
    if (ctl) {
      ctl->gamma = gamma;
      ctl->tau_B2 = xi_null_tau * s[0];
    }
  }
}

}  // namespace

hipError_t launch_control(Control* ctl, const double* part, const double* lam_part, int nblocks, double* ring,
                          double* dt_record, hipStream_t st) {
  hipLaunchKernelGGL(control_kernel, dim3(1), dim3(RT), 0, st, ctl, part, lam_part, nblocks, ring, dt_record);
  return hipGetLastError();
}

hipError_t launch_diag_finish(const double* part, int nblocks, double dV, double* out6, hipStream_t st) {
  hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(RT), 0, st, part, nblocks, dV, out6);
  return hipGetLastError();
}

hipError_t launch_begin_chunk(Control* ctl, int target, hipStream_t st) {
  hipLaunchKernelGGL(begin_chunk_kernel, dim3(1), dim3(64), 0, st, ctl, target);
  return hipGetLastError();
}

hipError_t launch_to_float(const double* src, float* dst, long long n, hipStream_t st) {
  long long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(to_float_kernel, dim3((unsigned)blocks), dim3(256), 0, st, src, dst, n);
  return hipGetLastError();
}

hipError_t launch_prescale(double* B0, long long N, const double scale[3], hipStream_t st) {
  long long blocks = (N + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(prescale_kernel, dim3((unsigned)blocks), dim3(256), 0, st, B0, N, scale[0], scale[1], scale[2]);
  return hipGetLastError();
}

hipError_t launch_max_norm2(const double* v, long long N, double* out, double* scratch, int nscratch,
                            hipStream_t st, Control* ctl, double gamma, double xi_null_tau) {
  long long blocks = (N + CT - 1) / CT;
  if (blocks > nscratch) blocks = nscratch;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(max_norm2_part_kernel, dim3((unsigned)blocks), dim3(CT), 0, st, v, N, scratch);
  hipLaunchKernelGGL(max_reduce_kernel, dim3(1), dim3(CT), 0, st, scratch, (int)blocks, out, ctl, gamma,
                     xi_null_tau);
  return hipGetLastError();
}

}  // namespace relax
