// 1-D wave equation for the vector potential of a normally incident,
// linearly polarised pulse (Sec. 5, Eq. Maxwell_ms):
//   (1/c^2) d^2A/dt^2 - d^2A/dX^2 = (4 pi / c) I(X, t),
// leapfrog in X and t with first-order Mur absorbing ends; the left end lets
// a prescribed incident wave in (the condition acts on A - A_inc). FP64.
#include "internal.h"

namespace td {

// interior update at point j
__device__ __forceinline__ double leap(const double* __restrict__ A_now, const double* __restrict__ A_prev,
                                       const double* __restrict__ I, int j, double S2, double src) {
  return 2.0 * A_now[j] - A_prev[j] + S2 * (A_now[j + 1] - 2.0 * A_now[j] + A_now[j - 1]) + src * I[j];
}

// One macroscopic step for all points. inc = (A_inc(X_0, t_n), A_inc(X_1, t_n),
// A_inc(X_0, t_{n+1}), A_inc(X_1, t_{n+1})). The end points recompute their
// inner neighbour's new value, so one launch suffices; I_old keeps this step's
// current for the work integral.
__global__ void k_fdtd_step(const double* __restrict__ A_now, const double* __restrict__ A_prev,
                            const double* __restrict__ I, double* __restrict__ A_new, double* __restrict__ I_old,
                            int n, double S2, double src, double q, double4 inc) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  I_old[j] = I[j];
  if (j > 0 && j < n - 1) {
    A_new[j] = leap(A_now, A_prev, I, j, S2, src);
  } else if (j == 0) {
    const double a1 = leap(A_now, A_prev, I, 1, S2, src);
    A_new[0] = inc.z + (A_now[1] - inc.y) + q * ((a1 - inc.w) - (A_now[0] - inc.x));
  } else {
    const double an = leap(A_now, A_prev, I, n - 2, S2, src);
    A_new[n - 1] = A_now[n - 2] + q * (an - A_now[n - 1]);
  }
}

// Append A(X_{x0+m}, t_n) / a_scale to each material point's window ring
// (FP32, [n_mat][W]) at slot `slot`.
__global__ void k_ring_push(const double* __restrict__ A, int x0, int n_mat, float* __restrict__ ring, int W,
                            int slot, double inv_scale) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_mat) return;
  ring[(size_t)m * W + slot] = (float)(A[x0 + m] * inv_scale);
}

// Causal windows from the rings: X[m][w] = ring[m][(head + 1 + w) mod W],
// oldest first, where `head` is the slot written last.
__global__ void k_ring_windows(const float* __restrict__ ring, int n_mat, int W, int head, float* __restrict__ X) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_mat * W) return;
  const int m = t / W, w = t - m * W;
  int s = head + 1 + w;
  if (s >= W) s -= W;
  X[t] = ring[(size_t)m * W + s];
}

// I(X_{x0+m}) = j_scale * y[m]; zero outside the material
__global__ void k_scatter_current(const float* __restrict__ y, int x0, int n_mat, int n, double j_scale,
                                  double* __restrict__ I) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int m = j - x0;
  I[j] = (m >= 0 && m < n_mat) ? j_scale * (double)y[m] : 0.0;
}

// amplitude gate of the surrogate: flag = 1 if |A| exceeds a_max at a medium
// point (every writer stores the same value)
__global__ void k_ms_gate(const double* __restrict__ A, int x0, int n_mat, double a_max, int* __restrict__ flag) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_mat) return;
  if (!(fabs(A[x0 + m]) <= a_max)) flag[0] = 1;
}

hipError_t launch_ms_gate(const double* A, int x0, int n_mat, double a_max, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_ms_gate, dim3((unsigned)((n_mat + 255) / 256)), dim3(256), 0, s, A, x0, n_mat, a_max, flag);
  return hipGetLastError();
}

hipError_t launch_fdtd_step(const double* A_now, const double* A_prev, const double* I, double* A_new,
                            double* I_old, int n, double S2, double src, double q, const double inc[4], hipStream_t s) {
  const double4 iv = make_double4(inc[0], inc[1], inc[2], inc[3]);
  hipLaunchKernelGGL(k_fdtd_step, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, A_now, A_prev, I, A_new,
                     I_old, n, S2, src, q, iv);
  return hipGetLastError();
}

hipError_t launch_ring_push(const double* A, int x0, int n_mat, float* ring, int W, int slot, double inv_scale,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_ring_push, dim3((unsigned)((n_mat + 255) / 256)), dim3(256), 0, s, A, x0, n_mat, ring, W,
                     slot, inv_scale);
  return hipGetLastError();
}

hipError_t launch_ring_windows(const float* ring, int n_mat, int W, int head, float* X, hipStream_t s) {
  const int n = n_mat * W;
  hipLaunchKernelGGL(k_ring_windows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, ring, n_mat, W, head, X);
  return hipGetLastError();
}

hipError_t launch_scatter_current(const float* y, int x0, int n_mat, int n, double j_scale, double* I,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_scatter_current, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, y, x0, n_mat, n,
                     j_scale, I);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Energy monitor of the coupled run (Sec. 5: the energy of the fields and of
// the electronic excitations together). Per unit area of the slab:
//   field: (1/8 pi) [sum_j E_j^2 + sum_links B^2] dX, E = -(A_now - A_prev)/(c dt)
//   (backward difference at every point), B = (A_{j+1} - A_j)/dX;
//   electrons: the work of the field, W += dt dX sum_m (I_m^n + I_m^{n+1})/2
//   E_m^{n+1/2} over the medium points (the excitation energy per area by the
//   work route of Sec. 4.1). One workgroup each, fixed-order sums.

__device__ __forceinline__ double block_sum_1024(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(1024) void k_em_energy(const double* __restrict__ A_now, const double* __restrict__ A_prev,
                                                    int n, double dx, double dt, double* __restrict__ out) {
  __shared__ double red[1024];
  const int t = threadIdx.x;
  double e2 = 0.0, b2 = 0.0;
  for (int j = t; j < n; j += 1024) {
    const double E = -(A_now[j] - A_prev[j]) / (kC * dt);
    e2 += E * E;
    if (j + 1 < n) {
      const double B = (A_now[j + 1] - A_now[j]) / dx;
      b2 += B * B;
    }
  }
  const double se = block_sum_1024(e2, red);
  const double sb = block_sum_1024(b2, red);
  if (t == 0) *out = (se + sb) * dx / (8.0 * M_PI);
}

// one macroscopic step's work over the medium points x0 .. x0 + n_mat - 1, and
// the step's records (each may be null): the medium points' histories hA, hI
// beside the sum, the rows A_row, I_row of all n points by the workgroups after
// the first, 1024 points each. A copy of its own for each was some 10 us of a
// step, its gap included; all by one workgroup, rows of 100000 points took
// longer than the copies (a step of the network 160 -> 196 us).
__global__ __launch_bounds__(1024) void k_ms_work_step(const double* __restrict__ A_new, const double* __restrict__ A_now,
                                                       const double* __restrict__ I_now, const double* __restrict__ I_new,
                                                       int n, int x0, int n_mat, double dx, double dt,
                                                       double* __restrict__ W, double* __restrict__ A_row,
                                                       double* __restrict__ I_row, double* __restrict__ hA,
                                                       double* __restrict__ hI) {
  __shared__ double red[1024];
  if (blockIdx.x > 0) {
    const int j = ((int)blockIdx.x - 1) * 1024 + (int)threadIdx.x;
    if (j < n && A_row) A_row[j] = A_new[j];
    if (j < n && I_row) I_row[j] = I_new[j];
    return;
  }
  double s = 0.0;
  for (int m = threadIdx.x; m < n_mat; m += 1024) {
    const int j = x0 + m;
    const double E = -(A_new[j] - A_now[j]) / (kC * dt);
    s += 0.5 * (I_now[j] + I_new[j]) * E;
    if (hA) hA[m] = A_new[j];
    if (hI) hI[m] = I_new[j];
  }
  const double tot = block_sum_1024(s, red);
  if (threadIdx.x == 0) *W += dt * dx * tot;
}

// the work from t_0 to t_steps from the medium histories A, I [(steps + 1)][n_mat]
__global__ __launch_bounds__(1024) void k_ms_work_history(const double* __restrict__ A, const double* __restrict__ I,
                                                          int steps, int n_mat, double dx, double dt,
                                                          double* __restrict__ W) {
  __shared__ double red[1024];
  double acc = 0.0;  // thread 0 keeps the running total
  for (int s = 0; s < steps; ++s) {
    double v = 0.0;
    for (int m = threadIdx.x; m < n_mat; m += 1024) {
      const size_t a = (size_t)s * n_mat + m, b = a + n_mat;
      const double E = -(A[b] - A[a]) / (kC * dt);
      v += 0.5 * (I[a] + I[b]) * E;
    }
    const double tot = block_sum_1024(v, red);
    acc += dt * dx * tot;
  }
  if (threadIdx.x == 0) *W = acc;
}

hipError_t launch_em_energy(const double* A_now, const double* A_prev, int n, double dx, double dt, double* out,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_em_energy, dim3(1), dim3(1024), 0, s, A_now, A_prev, n, dx, dt, out);
  return hipGetLastError();
}

hipError_t launch_ms_work_step(const double* A_new, const double* A_now, const double* I_now, const double* I_new,
                               int n, int x0, int n_mat, double dx, double dt, double* W, double* A_row,
                               double* I_row, double* hA, double* hI, hipStream_t s) {
  const unsigned rows = A_row || I_row ? (unsigned)((n + 1023) / 1024) : 0;
  hipLaunchKernelGGL(k_ms_work_step, dim3(1 + rows), dim3(1024), 0, s, A_new, A_now, I_now, I_new, n, x0, n_mat, dx, dt, W,
                     A_row, I_row, hA, hI);
  return hipGetLastError();
}

hipError_t launch_ms_work_history(const double* A, const double* I, int steps, int n_mat, double dx, double dt,
                                  double* W, hipStream_t s) {
  hipLaunchKernelGGL(k_ms_work_history, dim3(1), dim3(1024), 0, s, A, I, steps, n_mat, dx, dt, W);
  return hipGetLastError();
}

}  // namespace td
