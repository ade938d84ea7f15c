// Kernels of the batched path: several independent registration problems of
// different sizes advance together, one launch per phase.  Problem tables sit
// in kernel-argument memory (uniform, scalar loads); each problem keeps its
// own float64 partial sums in the same block layout as a single-problem
// launch, so sums (and results) equal the single-problem path bit for bit.
//
// The conjugate-gradient iteration (Sec. 2.3.1) is steered on the device:
// per problem an active flag, iteration count, status and relative residual
// live in device memory, so a fixed sequence of launches can be captured once
// into a HIP graph and replayed; finished problems turn into no-ops.
#include "mfr_internal.h"

namespace mfr {

namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sred) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) sred[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += sred[w];
  }
  __syncthreads();
  return s;
}

template <int N>
__device__ __forceinline__ int find_job(const int (&prefix)[N], int n, int item) {
  int j = 0;
  while (j + 1 < n && prefix[j + 1] <= item) ++j;
  return j;
}

}  // namespace

// ---- per-problem fixed-order sums: one group per problem -------------------------
// (the order of launch_sum, so that both give the same bits)
__global__ __launch_bounds__(1024) void sum_batch_kernel(const SumJobs J) {
  __shared__ double sred[16];
  const SumJob& s = J.jobs[blockIdx.x];
  if (J.active && !ld_coherent(J.active + blockIdx.x)) return;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  int i = threadIdx.x;
  for (; i + 3 * 1024 < s.n; i += 4 * 1024) {
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] += s.parts[(i + k * 1024) * s.stride];
  }
  for (; i < s.n; i += 1024) a[0] += s.parts[i * s.stride];
  const double t = block_sum<1024>((a[0] + a[1]) + (a[2] + a[3]), sred);
  if (threadIdx.x == 0) *s.out = t;
}

hipError_t launch_sum_batch(const SumJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(sum_batch_kernel, dim3(j.n), dim3(1024), 0, st, j);
  return hipGetLastError();
}

// ---- batched vector kernels ------------------------------------------------------
// y_j = x_j + eta_j s_j for active problems
__global__ __launch_bounds__(kVecBlock) void axpy_batch_kernel(const AxpyJobs J) {
  const int pr = find_job(J.prefix, J.n, blockIdx.x);
  if (J.active && !ld_coherent(J.active + pr)) return;
  const AxpyJob& a = J.jobs[pr];
  const int nb = J.prefix[pr + 1] - J.prefix[pr];
  for (int i = (blockIdx.x - J.prefix[pr]) * kVecBlock + threadIdx.x; i < a.n; i += nb * kVecBlock)
    a.y[i] = fmaf(a.eta, a.s[i], a.x[i]);
}

hipError_t launch_axpy_batch(const AxpyJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(axpy_batch_kernel, dim3(j.prefix[j.n]), dim3(kVecBlock), 0, st, j);
  return hipGetLastError();
}

// x_j . y_j partials (one per block of the problem, same layout as launch_dot)
__global__ __launch_bounds__(kVecBlock) void dot_batch_kernel(const VecJobs J) {
  __shared__ double sred[kVecBlock / 64];
  const int pr = find_job(J.prefix, J.n, blockIdx.x);
  const VecJob& v = J.jobs[pr];
  const int lb = blockIdx.x - J.prefix[pr], nb = J.prefix[pr + 1] - J.prefix[pr];
  double a = 0.0;
  for (int i = lb * kVecBlock + threadIdx.x; i < v.n3; i += nb * kVecBlock) a += (double)v.r[i] * v.z[i];
  const double s = block_sum<kVecBlock>(a, sred);
  if (threadIdx.x == 0) v.red[lb] = s;
}

hipError_t launch_dot_batch(const VecJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(dot_batch_kernel, dim3(j.prefix[j.n]), dim3(kVecBlock), 0, st, j);
  return hipGetLastError();
}

// PCG start: s = 0, r = b, z = M^-1 r, p = z; partials (b.b, r.z); state reset.
__global__ __launch_bounds__(kVecBlock) void pcg_init_batch_kernel(const VecJobs J) {
  __shared__ double sred[kVecBlock / 64];
  const int pr = find_job(J.prefix, J.n, blockIdx.x);
  const VecJob& v = J.jobs[pr];
  const int lb = blockIdx.x - J.prefix[pr], nb = J.prefix[pr + 1] - J.prefix[pr];
  double bb = 0.0, rz = 0.0;
  for (int i = lb * kVecBlock + threadIdx.x; i < v.n3; i += nb * kVecBlock) {
    const float bi = v.b[i];
    const float zi = v.diag ? bi / v.diag[i] : bi;
    v.s[i] = 0.0f;
    v.r[i] = bi;
    v.z[i] = zi;
    v.p[i] = zi;
    bb += (double)bi * bi;
    rz += (double)bi * zi;
  }
  const double sb = block_sum<kVecBlock>(bb, sred);
  const double sz = block_sum<kVecBlock>(rz, sred);
  if (threadIdx.x == 0) {
    v.red[2 * lb] = sb;
    v.red[2 * lb + 1] = sz;
  }
}

// One group per problem: ||b||, r.z, and the per-problem control state.
__global__ __launch_bounds__(256) void pcg_init_finish_batch_kernel(const VecJobs J) {
  __shared__ double sred[4];
  const int pr = blockIdx.x;
  const VecJob& v = J.jobs[pr];
  const int nb = J.prefix[pr + 1] - J.prefix[pr];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) {
    a += v.red[2 * i];
    b += v.red[2 * i + 1];
  }
  const double bb = block_sum<256>(a, sred);
  const double rz = block_sum<256>(b, sred);
  if (threadIdx.x == 0) {
    double* sc = v.sc;
    sc[SC_BB] = bb;
    sc[SC_RZ] = rz;
    sc[SC_RR] = bb;
    sc[SC_RELRES] = (bb > 0.0) ? 1.0 : 0.0;
    int* st = v.state;
    const bool live = bb > 0.0 && isfinite(bb) && v.max_iter > 0;
    st[ST_ITERS] = 0;
    st[ST_MAXIT] = v.max_iter;
    st[ST_FALLBACK] = 0;
    sc[SC_RTOL] = v.rtol;
    st[ST_FLAG] = (bb == 0.0) ? 0 : 1;
    st[ST_ACTIVE] = live ? 1 : 0;
    J.active_out[pr] = live ? 1 : 0;
  }
}

// The result of a device-steered solve into caller memory: {iterations,
// relative residual, flag} (the capturable solve).
__global__ void pcg_info_out_kernel(const int* __restrict__ state, const double* __restrict__ sc,
                                    double* __restrict__ out) {
  if (threadIdx.x != 0) return;
  out[0] = (double)state[ST_ITERS];
  out[1] = sc[SC_RELRES];
  out[2] = (double)state[ST_FLAG];
}

hipError_t launch_pcg_info_out(const int* state, const double* sc, double* out, hipStream_t st) {
  hipLaunchKernelGGL(pcg_info_out_kernel, dim3(1), dim3(64), 0, st, state, sc, out);
  return hipGetLastError();
}

hipError_t launch_pcg_init_batch(const VecJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(pcg_init_batch_kernel, dim3(j.prefix[j.n]), dim3(kVecBlock), 0, st, j);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pcg_init_finish_batch_kernel, dim3(j.n), dim3(256), 0, st, j);
  return hipGetLastError();
}

// alpha = r.z / p.q from the node-pass partials (flexible solve); breakdown ends the problem.
// One 1024-thread group per problem with two independent running sums per thread
// (a fixed order, so the result does not depend on timing).
__global__ __launch_bounds__(1024) void pcg_alpha_batch_kernel(const VecJobs J) {
  __shared__ double sred[16];
  const int pr = blockIdx.x;
  const VecJob& v = J.jobs[pr];
  if (!ld_coherent(v.state + ST_ACTIVE)) return;
  double a = 0.0, b = 0.0;
  int i = threadIdx.x;
  for (; i + 1024 < v.n_pq; i += 2048) {
    a += v.red_pq[i];
    b += v.red_pq[i + 1024];
  }
  if (i < v.n_pq) a += v.red_pq[i];
  const double pq = block_sum<1024>(a + b, sred);
  if (threadIdx.x == 0) {
    double* sc = v.sc;
    sc[SC_PQ] = pq;
    if (pq > 0.0 && isfinite(pq)) {
      sc[SC_ALPHA] = ld_coherent(sc + SC_RZ) / pq;
    } else {
      sc[SC_ALPHA] = 0.0;
      v.state[ST_FLAG] = 2;
      v.state[ST_ACTIVE] = 0;
      J.active_out[pr] = 0;
    }
  }
}

hipError_t launch_pcg_alpha_batch(const VecJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(pcg_alpha_batch_kernel, dim3(j.n), dim3(1024), 0, st, j);
  return hipGetLastError();
}

// ---- one CG iteration after the node pass: two launches --------------------------
// Every group sums the partials of the preceding kernel itself (at most kNodeGroups
// or 2 x 1024 float64 values, read through L2) in the same fixed order, so all of
// them hold the same alpha (beta) and the same verdict, and the first group of a
// problem writes the scalars and the control state.  The kernels with one group per
// problem that formed alpha and beta took 4.5 us each, plus their launch gaps, for
// a few hundred additions.  Nothing that the update's groups read is written in its
// launch: a breakdown it finds ends the solve in the step kernel, which sees it from
// the stored p.q.  There the first group clears the active flag while others start,
// so one thread reads the flag for its whole group: waves that each read it could
// part, and those left would sum without the others' share.  A group that finds the
// flag cleared has nothing to do: the solve is over and its p is not used any more.
__device__ __forceinline__ double sum_parts(const double* __restrict__ parts, int n, double* sred, double* stot) {
  double a = 0.0, b = 0.0;
  int i = threadIdx.x;
  for (; i + kVecBlock < n; i += 2 * kVecBlock) {
    a += parts[i];
    b += parts[i + kVecBlock];
  }
  if (i < n) a += parts[i];
  const double s = block_sum<kVecBlock>(a + b, sred);
  if (threadIdx.x == 0) *stot = s;
  __syncthreads();
  return *stot;
}

// A breakdown: p.q <= 0 or not finite.
__device__ __forceinline__ bool pq_ok(double pq) { return pq > 0.0 && isfinite(pq); }

// alpha = r.z / p.q; s += alpha p, r -= alpha q, z = M^-1 r (none of these after a
// breakdown); partials of r.r and r.z.
__global__ __launch_bounds__(kVecBlock) void pcg_update_batch_kernel(const VecJobs J) {
  __shared__ double sred[kVecBlock / 64], stot;
  const int pr = find_job(J.prefix, J.n, blockIdx.x);
  const VecJob& v = J.jobs[pr];
  if (!ld_coherent(v.state + ST_ACTIVE)) return;
  const int lb = blockIdx.x - J.prefix[pr], nb = J.prefix[pr + 1] - J.prefix[pr];
  const double rz_old = ld_coherent(v.sc + SC_RZ);
  const double pq = sum_parts(v.red_pq, v.n_pq, sred, &stot);
  const bool ok = pq_ok(pq);
  const double alpha_d = ok ? rz_old / pq : 0.0;
  if (lb == 0 && threadIdx.x == 0) {
    double* sc = v.sc;
    sc[SC_PQ] = pq;
    sc[SC_ALPHA] = alpha_d;
    sc[SC_RZOLD] = rz_old;
    v.state[ST_NEXT] = ld_coherent(v.state + ST_ITERS) + 1;
  }
  if (!ok) return;
  const float alpha = (float)alpha_d;
  double rr = 0.0, rz = 0.0;
  for (int i = lb * kVecBlock + threadIdx.x; i < v.n3; i += nb * kVecBlock) {
    const float ri = fmaf(-alpha, v.q[i], v.r[i]);
    v.s[i] = fmaf(alpha, v.p[i], v.s[i]);
    v.r[i] = ri;
    const float zi = v.diag ? ri / v.diag[i] : ri;
    v.z[i] = zi;
    rr += (double)ri * ri;
    rz += (double)ri * zi;
  }
  const double a = block_sum<kVecBlock>(rr, sred);
  const double b = block_sum<kVecBlock>(rz, sred);
  if (threadIdx.x == 0) {
    v.red[lb] = a;
    v.red[nb + lb] = b;
  }
}

hipError_t launch_pcg_update_batch(const VecJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(pcg_update_batch_kernel, dim3(j.prefix[j.n]), dim3(kVecBlock), 0, st, j);
  return hipGetLastError();
}

// |r|, beta = (r.z)_new / (r.z)_old and the convergence test; p = z + beta p unless
// the solve has stopped.  After a breakdown it only ends the solve.
__global__ __launch_bounds__(kVecBlock) void pcg_step_batch_kernel(const VecJobs J) {
  __shared__ double sred[kVecBlock / 64], stot;
  __shared__ int sgo;   // 0: stopped before this launch or already by it; 1: go on; 2: breakdown
  const int pr = find_job(J.prefix, J.n, blockIdx.x);
  const VecJob& v = J.jobs[pr];
  if (threadIdx.x == 0) {
    const double pq = ld_coherent(v.sc + SC_PQ);
    sgo = !ld_coherent(v.state + ST_ACTIVE) ? 0 : pq_ok(pq) ? 1 : 2;
  }
  __syncthreads();
  const int go = sgo;
  const int lb = blockIdx.x - J.prefix[pr], nb = J.prefix[pr + 1] - J.prefix[pr];
  if (go == 2 && lb == 0 && threadIdx.x == 0) {
    v.state[ST_FLAG] = 2;
    v.state[ST_ACTIVE] = 0;
    J.active_out[pr] = 0;
  }
  if (go != 1) return;
  const double rr = sum_parts(v.red, nb, sred, &stot);
  __syncthreads();
  const double rz = sum_parts(v.red + nb, nb, sred, &stot);
  const double rz_old = ld_coherent(v.sc + SC_RZOLD), bb = ld_coherent(v.sc + SC_BB), rtol = ld_coherent(v.sc + SC_RTOL);
  const int iters = ld_coherent(v.state + ST_NEXT), maxit = ld_coherent(v.state + ST_MAXIT);
  const double beta = rz / rz_old, rel = sqrt(rr) / sqrt(bb);
  const bool done = rel <= rtol || iters >= maxit;
  if (lb == 0 && threadIdx.x == 0) {
    double* sc = v.sc;
    int* st = v.state;
    sc[SC_RR] = rr;
    sc[SC_RZNEW] = rz;
    sc[SC_BETA] = beta;
    sc[SC_RZ] = rz;
    sc[SC_RELRES] = rel;
    st[ST_ITERS] = iters;
    if (done) {
      st[ST_FLAG] = rel <= rtol ? 0 : 1;
      st[ST_ACTIVE] = 0;
    }
    J.active_out[pr] = done ? 0 : 1;
  }
  if (done) return;
  const float b = (float)beta;
  for (int i = lb * kVecBlock + threadIdx.x; i < v.n3; i += nb * kVecBlock) v.p[i] = fmaf(b, v.p[i], v.z[i]);
}

hipError_t launch_pcg_step_batch(const VecJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(pcg_step_batch_kernel, dim3(j.prefix[j.n]), dim3(kVecBlock), 0, st, j);
  return hipGetLastError();
}

// p = z + beta p with the beta of the flexible solve
__global__ __launch_bounds__(kVecBlock) void pcg_direction_batch_kernel(const VecJobs J) {
  const int pr = find_job(J.prefix, J.n, blockIdx.x);
  const VecJob& v = J.jobs[pr];
  if (!ld_coherent(v.state + ST_ACTIVE)) return;
  const int lb = blockIdx.x - J.prefix[pr], nb = J.prefix[pr + 1] - J.prefix[pr];
  const float beta = (float)ld_coherent(v.sc + SC_BETA);
  for (int i = lb * kVecBlock + threadIdx.x; i < v.n3; i += nb * kVecBlock) v.p[i] = fmaf(beta, v.p[i], v.z[i]);
}

hipError_t launch_pcg_direction_batch(const VecJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(pcg_direction_batch_kernel, dim3(j.prefix[j.n]), dim3(kVecBlock), 0, st, j);
  return hipGetLastError();
}

}  // namespace mfr
