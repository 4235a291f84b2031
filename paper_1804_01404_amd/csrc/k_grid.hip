// Grid-side kernels of one time step: per-step field parameters, the density
// (Eq. rho), the Hartree potential by FFT (periodic 4 pi / G^2; isolated
// free-space convolution on a doubled box), the adiabatic PZ81 LDA (Sec. 3.1),
// the macroscopic current reduction (Eq. macro_current) and the step counter.
// Every reduction runs in a fixed order, so two runs give identical bits.
#include "internal.h"

namespace td {

// ---------------------------------------------------------------- step begin
// A: table [..][3]; the step index n is *counter (or 0). Velocity gauge:
// kappa = k + (A_n + A_{n+1}) / (2c), kappaJ = k + A_{n+1} / c, and the
// matching sphere phases exp(i A.x / c). Length gauge: kappa = kappaJ = k,
// unit phases, E_n = -(A_{n+1} - A_n) / (c dt). With coef, also the k-point
// rows of stencil coefficients in the stage precision (-1/2 c_m / h_mu^2 and
// kappa_mu d_m / h_mu per axis, the diagonal -1/2 sum_mu c_0 / h_mu^2 +
// |kappa|^2 / 2); with phkA, exp(i kappa . x_e) for every k-point and entry.
// One launch: as three (field, coefficients, phases) of about 4.5 us each they
// were a tenth of a small cell's step. A workgroup takes 256 entries and
// kBeginK k-points, and forms its entries' A phases anew (a sincos or two).
constexpr int kBeginK = 8;

template <typename T>
__device__ __forceinline__ void step_begin_block(const ParamCell& c, int bx, int by) {
  const double* A0 = c.A + 3 * (size_t)(c.counter ? *c.counter : 0);
  const double* A1 = A0 + 3;
  const bool vel = (c.gauge == 0);
  double ab[3], a1[3];
  for (int i = 0; i < 3; ++i) {
    ab[i] = 0.5 * (A0[i] + A1[i]);
    a1[i] = A1[i];
  }
  const int t = threadIdx.x;
  const int k0 = by * kBeginK, k1 = min(c.n_k, k0 + kBeginK);
  if (bx == 0) {
    if (by == 0 && t < 3) {
      c.efield[t] = vel ? 0.0 : -(A1[t] - A0[t]) / (kC * c.dt);
      c.Alast[t] = A1[t];
    }
    // 32 threads per k-point: 25 coefficients, kappa, kappaJ
    const int k = k0 + t / 32, j = t % 32;
    if (k < k1) {
      double kap[3];
      for (int i = 0; i < 3; ++i) kap[i] = c.kpt[3 * k + i] + (vel ? ab[i] / kC : 0.0);
      if (j >= 25) {
        const int i = (j - 25) % 3;
        if (j < 28)
          c.kappa[3 * k + i] = kap[i];
        else if (j < 31)
          c.kappaJ[3 * k + i] = c.kpt[3 * k + i] + (vel ? a1[i] / kC : 0.0);
      } else if (c.coef) {
        const int mu = j / 8, m = j % 4;
        double v;
        if (j == kCoefDiag)
          v = c.cdiag + 0.5 * (kap[0] * kap[0] + kap[1] * kap[1] + kap[2] * kap[2]);
        else
          v = j % 8 < kCoefB ? c.lap[mu][m + 1] : kap[mu] * c.dh[mu][m];
        static_cast<T*>(c.coef)[(size_t)k * kCoef + j] = (T)v;
      }
    }
  }
  const int e = bx * blockDim.x + t;
  if (e >= c.S) return;
  double2 ph = make_double2(1.0, 0.0), phj = ph;
  if (vel) {
    const double* x = c.ent_x + 3 * (size_t)e;
    double sn, cs;
    sincos((ab[0] * x[0] + ab[1] * x[1] + ab[2] * x[2]) / kC, &sn, &cs);
    ph = make_double2(cs, sn);
    if (by == 0) {
      sincos((a1[0] * x[0] + a1[1] * x[1] + a1[2] * x[2]) / kC, &sn, &cs);
      phj = make_double2(cs, sn);
    }
  }
  if (by == 0) {
    c.phA[e] = ph;
    c.phAJ[e] = phj;
  }
  if (c.phkA) {
    for (int k = k0; k < k1; ++k) {
      const double2 p1 = c.phk[(size_t)k * c.S + e];
      c.phkA[(size_t)k * c.S + e] = make_double2(p1.x * ph.x - p1.y * ph.y, p1.x * ph.y + p1.y * ph.x);
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_step_begin(ParamCell c) {
  step_begin_block<T>(c, (int)blockIdx.x, (int)blockIdx.y);
}

// the same for the cells of a group (cell blockIdx.z), each at its own step;
// the group's work queue starts over
template <typename T>
__global__ __launch_bounds__(256) void k_step_begin_group(const ParamCell* __restrict__ tab, int* queue) {
  if (blockIdx.x + blockIdx.y + blockIdx.z == 0 && threadIdx.x == 0) *queue = 0;
  const ParamCell& c = tab[blockIdx.z];
  if ((int)blockIdx.x > 0 && (int)blockIdx.x * 256 >= c.S) return;
  if ((int)blockIdx.y * kBeginK >= c.n_k) return;
  step_begin_block<T>(c, (int)blockIdx.x, (int)blockIdx.y);
}

template <typename T>
hipError_t launch_step_begin(const ParamCell& c, hipStream_t s) {
  const dim3 grid((unsigned)max(1, (c.S + 255) / 256), (unsigned)((c.n_k + kBeginK - 1) / kBeginK));
  hipLaunchKernelGGL((k_step_begin<T>), grid, dim3(256), 0, s, c);
  return hipGetLastError();
}
template hipError_t launch_step_begin<double>(const ParamCell&, hipStream_t);
template hipError_t launch_step_begin<float>(const ParamCell&, hipStream_t);

template <typename T>
hipError_t launch_step_begin_group(const ParamCell* tab, int ncells, int max_S, int max_nk, int* queue,
                                   hipStream_t s) {
  const dim3 grid((unsigned)max(1, (max_S + 255) / 256), (unsigned)((max_nk + kBeginK - 1) / kBeginK),
                  (unsigned)ncells);
  hipLaunchKernelGGL((k_step_begin_group<T>), grid, dim3(256), 0, s, tab, queue);
  return hipGetLastError();
}
template hipError_t launch_step_begin_group<double>(const ParamCell*, int, int, int, int*, hipStream_t);
template hipError_t launch_step_begin_group<float>(const ParamCell*, int, int, int, int*, hipStream_t);

// ---------------------------------------------------------------- batch tables
__global__ void k_batch_tables_in(const IOCell* __restrict__ io, const double* __restrict__ staged, int len) {
  const IOCell& c = io[blockIdx.x];
  const double* src = staged + (size_t)blockIdx.x * len;
  for (int i = threadIdx.x; i < len; i += blockDim.x) c.A[i] = src[i];
  if (threadIdx.x == 0) *c.counter = 0;
}

__global__ void k_batch_tables_out(const IOCell* __restrict__ io, double* __restrict__ staged, int len) {
  const IOCell& c = io[blockIdx.x];
  double* dst = staged + (size_t)blockIdx.x * (len + 1);
  for (int i = threadIdx.x; i < len; i += blockDim.x) dst[i] = c.J[i];
  if (threadIdx.x == 0) dst[len] = (double)*c.nanflag;
}

hipError_t launch_batch_tables_in(const IOCell* io, int ncells, const double* staged, int len, hipStream_t s) {
  if (ncells <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_tables_in, dim3(ncells), dim3(64), 0, s, io, staged, len);
  return hipGetLastError();
}

hipError_t launch_batch_tables_out(const IOCell* io, int ncells, double* staged, int len, hipStream_t s) {
  if (ncells <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_tables_out, dim3(ncells), dim3(64), 0, s, io, staged, len);
  return hipGetLastError();
}

// ---------------------------------------------------------------- finish
// One workgroup (256 threads at work): I = -(1/Omega) sum_o f_o [p_o + kappaJ_k norm_o + jNL_o],
// the orbital energy sum_o f_o [kin + kappaJ.p + 1/2 |kappaJ|^2 norm + vloc + E_NL],
// and the occupied norm; f_o = 2 w_k. Thread t sums orbitals t, t + 256, ...
// in order, then a fixed pairwise tree combines the threads. nanflag gets
// bit 0 for a non-finite norm or momentum, bit 1 (only when norm_tol > 0)
// for a norm further than norm_tol from 1.
constexpr int kFinishThreads = 256;

__device__ __forceinline__ void finish_block(const TailCell& c, int bump, double (*red)[5]) {
  const int t = threadIdx.x;
  const int n_tot = c.n_orb * c.n_k, tiles = c.tiles;
  double cx = 0, cy = 0, cz = 0, en = 0, nr = 0;
  int bad = 0;
  for (int o = t < kFinishThreads ? t : n_tot; o < n_tot; o += kFinishThreads) {
    const int k = o / c.n_orb;
    double s[6] = {0, 0, 0, 0, 0, 0};
    for (int tl = 0; tl < tiles; ++tl)
      for (int i = 0; i < 6; ++i) s[i] += c.obs[((size_t)o * tiles + tl) * 8 + i];
    for (int i = 0; i < 6; ++i) s[i] *= c.dV;
    const double f = 2.0 * c.kw[k];
    const double kx = c.kappaJ[3 * k], ky = c.kappaJ[3 * k + 1], kz = c.kappaJ[3 * k + 2];
    double jx = 0, jy = 0, jz = 0, enl = 0;
    if (c.use_nl) {
      jx = c.jnl[4 * (size_t)o];
      jy = c.jnl[4 * (size_t)o + 1];
      jz = c.jnl[4 * (size_t)o + 2];
      enl = c.jnl[4 * (size_t)o + 3];
    }
    cx += f * (s[1] + kx * s[0] + jx);
    cy += f * (s[2] + ky * s[0] + jy);
    cz += f * (s[3] + kz * s[0] + jz);
    en += f * (s[4] + kx * s[1] + ky * s[2] + kz * s[3] + 0.5 * (kx * kx + ky * ky + kz * kz) * s[0] +
               s[5] + enl);
    nr += f * s[0];
    if (!isfinite(s[0]) || !isfinite(s[1]) || !isfinite(s[2]) || !isfinite(s[3])) bad |= 1;
    else if (c.norm_tol > 0.0 && fabs(s[0] - 1.0) > c.norm_tol) bad |= 2;
  }
  if (t < kFinishThreads) {
    red[t][0] = cx;
    red[t][1] = cy;
    red[t][2] = cz;
    red[t][3] = en;
    red[t][4] = nr;
  }
  __syncthreads();
  for (int w = kFinishThreads / 2; w > 0; w >>= 1) {
    if (t < w)
      for (int i = 0; i < 5; ++i) red[t][i] += red[t + w][i];
    __syncthreads();
  }
  if (bad) atomicOr(c.nanflag, bad);
  if (t == 0) {
    const double J[3] = {-red[0][0] / c.volume, -red[0][1] / c.volume, -red[0][2] / c.volume};
    for (int i = 0; i < 3; ++i) c.scalars[i] = J[i];
    c.scalars[3] = red[0][3];
    c.scalars[4] = red[0][4];
    if (bump) {
      const int n = *c.counter;
      for (int i = 0; i < 3; ++i) c.Jtab[3 * (size_t)n + i] = J[i];
      *c.counter = n + 1;
    }
  }
}

__global__ __launch_bounds__(kFinishThreads) void k_finish(TailCell c, int bump) {
  __shared__ double red[kFinishThreads][5];
  finish_block(c, bump, red);
}

hipError_t launch_finish(const TailCell& c, int bump, hipStream_t s) {
  hipLaunchKernelGGL(k_finish, dim3(1), dim3(kFinishThreads), 0, s, c, bump);
  return hipGetLastError();
}

// ---------------------------------------------------------------- density
// part[c][p] = sum over orbitals o in chunk c of 2 w_k |w_o(p)|^2, in order.
// The loads of kRhoPipe orbitals are issued together: one by one a thread
// waits out the memory latency per orbital (20.8 us for the 16 cells of 64
// orbitals of a 12^3 slab, 14 MB).
constexpr int kRhoPipe = 8;

template <typename T>
__device__ __forceinline__ void rho_partial_point(const TailCell& t, int N, int c, int p) {
  const auto* __restrict__ w = static_cast<const typename Vec2<T>::type*>(t.w) + p;
  const int n_tot = t.n_orb * t.n_k;
  const int o0 = c * t.chunk, o1 = min(n_tot, o0 + t.chunk);
  double acc = 0.0;
  for (int o = o0; o < o1; o += kRhoPipe) {
    typename Vec2<T>::type v[kRhoPipe];
#pragma unroll
    for (int u = 0; u < kRhoPipe; ++u) v[u] = w[(size_t)min(o + u, o1 - 1) * N];
#pragma unroll
    for (int u = 0; u < kRhoPipe; ++u) {
      const double re = (double)v[u].x, im = (double)v[u].y;
      if (o + u < o1) acc += 2.0 * t.kw[(o + u) / t.n_orb] * (re * re + im * im);
    }
  }
  t.rho_out[(size_t)c * N + p] = acc;
}

// with_finish: the first workgroup forms the current instead (it needs the
// observables only, and is over long before the density pass)
template <typename T>
__device__ __forceinline__ void density_block(const TailCell& t, int N, int with_finish, int bump, int b) {
  __shared__ double red[kFinishThreads][5];
  if (with_finish && b == 0) {
    finish_block(t, bump, red);
    return;
  }
  b -= with_finish;
  const int bpc = (N + 255) / 256;
  const int c = b / bpc, p = (b - c * bpc) * 256 + (int)threadIdx.x;
  if (c < t.nchunks && p < N) rho_partial_point<T>(t, N, c, p);
}

template <typename T>
__global__ __launch_bounds__(256) void k_density(TailCell t, int N, int with_finish) {
  density_block<T>(t, N, with_finish, 1, (int)blockIdx.x);
}

// the same for the cells of a group (cell blockIdx.y)
template <typename T>
__global__ __launch_bounds__(256) void k_density_group(const TailCell* __restrict__ tab, int N) {
  density_block<T>(tab[blockIdx.y], N, 1, 1, (int)blockIdx.x);
}

// Orbitals per chunk: enough (chunk, point block) workgroups to fill the chip
// (about 2048), but at least 16 orbitals, so that the partial planes stay
// under a tenth of the orbitals' bytes, and at most 128.
int density_chunk(int N, int n_tot) {
  const long want = (long)n_tot * ((N + 255) / 256) / 2048;
  return (int)std::max(16L, std::min(128L, want));
}

template <typename T>
hipError_t launch_density(const TailCell& t, int N, int with_finish, hipStream_t s) {
  const unsigned grid = (unsigned)(with_finish + (N + 255) / 256 * t.nchunks);
  hipLaunchKernelGGL((k_density<T>), dim3(grid), dim3(256), 0, s, t, N, with_finish);
  return hipGetLastError();
}
template hipError_t launch_density<double>(const TailCell&, int, int, hipStream_t);
template hipError_t launch_density<float>(const TailCell&, int, int, hipStream_t);

template <typename T>
hipError_t launch_density_group(const TailCell* tab, int ncells, int N, int max_chunks, hipStream_t s) {
  const dim3 grid((unsigned)(1 + (N + 255) / 256 * max_chunks), (unsigned)ncells);
  hipLaunchKernelGGL((k_density_group<T>), grid, dim3(256), 0, s, tab, N);
  return hipGetLastError();
}
template hipError_t launch_density_group<double>(const TailCell*, int, int, int, hipStream_t);
template hipError_t launch_density_group<float>(const TailCell*, int, int, int, hipStream_t);

// rho[p] = sum over chunks of part[c][p]. A workgroup takes 64 points and
// kRedSlices slices: slice j sums chunks j, j + kRedSlices, ... in order, then
// the slices combine by a fixed pairwise tree in LDS, so the result does not
// depend on scheduling. One thread per point looping over every chunk would
// leave the chip nearly idle (8000 points are 32 workgroups) behind a chain
// of dependent loads.
constexpr int kRedSlices = 16;

__device__ __forceinline__ void rho_reduce_block(const double* __restrict__ part, int nchunks, int N,
                                                 double* __restrict__ rho, int b, double (*red)[64]) {
  const int i = threadIdx.x & 63, j = threadIdx.x >> 6;
  const int p = b * 64 + i;
  double acc = 0.0;
  if (p < N)
    for (int c = j; c < nchunks; c += kRedSlices) acc += part[(size_t)c * N + p];
  red[j][i] = acc;
  __syncthreads();
  for (int h = kRedSlices / 2; h > 0; h >>= 1) {
    if (j < h) red[j][i] += red[j + h][i];
    __syncthreads();
  }
  if (j == 0 && p < N) rho[p] = red[0][i];
}

__global__ __launch_bounds__(64 * kRedSlices) void k_rho_reduce(const double* __restrict__ part, int nchunks,
                                                                int N, double* __restrict__ rho) {
  __shared__ double red[kRedSlices][64];
  rho_reduce_block(part, nchunks, N, rho, (int)blockIdx.x, red);
}

// rho and tau in one launch, with the current of the step on its first
// workgroup (with_finish): three launches of 5 to 6 us on a 20^3 cell
__global__ __launch_bounds__(64 * kRedSlices) void k_rho_tau_reduce(TailCell t, int N, const double* tau_part,
                                                                    double* tau, int with_finish) {
  __shared__ double red[kFinishThreads * 5];
  int b = (int)blockIdx.x;
  if (with_finish && b == 0) {
    finish_block(t, 1, reinterpret_cast<double(*)[5]>(red));
    return;
  }
  b -= with_finish;
  const int nb = (N + 63) / 64;
  const bool second = b >= nb;
  rho_reduce_block(second ? tau_part : t.rho_part, t.nchunks, N, second ? tau : t.rho, second ? b - nb : b,
                   reinterpret_cast<double(*)[64]>(red));
}

// the same for the cells of a group (cell blockIdx.y; cells with one chunk
// have their density already)
__global__ __launch_bounds__(64 * kRedSlices) void k_rho_reduce_group(const TailCell* __restrict__ tab, int N) {
  __shared__ double red[kRedSlices][64];
  const TailCell& t = tab[blockIdx.y];
  if (t.nchunks <= 1) return;
  rho_reduce_block(t.rho_part, t.nchunks, N, t.rho, (int)blockIdx.x, red);
}

hipError_t launch_rho_tau_reduce(const TailCell& t, int N, const double* tau_part, double* tau, int with_finish,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_rho_tau_reduce, dim3((unsigned)(with_finish + 2 * ((N + 63) / 64))), dim3(64 * kRedSlices), 0,
                     s, t, N, tau_part, tau, with_finish);
  return hipGetLastError();
}

hipError_t launch_rho_reduce_group(const TailCell* tab, int ncells, int N, hipStream_t s) {
  hipLaunchKernelGGL(k_rho_reduce_group, dim3((N + 63) / 64, ncells), dim3(64 * kRedSlices), 0, s, tab, N);
  return hipGetLastError();
}

hipError_t launch_rho_reduce(const double* part, int nchunks, int N, double* rho, hipStream_t s) {
  hipLaunchKernelGGL(k_rho_reduce, dim3((N + 63) / 64), dim3(64 * kRedSlices), 0, s, part, nchunks, N, rho);
  return hipGetLastError();
}

// ---------------------------------------------------------------- FFT
// In-place FP64 complex FFT of lines along one axis of an M1 x M2 x M3 array
// (M1 fastest), unnormalised, sign -1 forward / +1 inverse. A workgroup
// stages B lines in LDS and runs a Stockham mixed-radix (8, 4, 2, 3, 5)
// transform: for radix R and Ns = product of the radices already applied,
// butterfly j reads in[j + r M/R], multiplies by exp(sign 2 pi i r (j mod Ns) / (Ns R)),
// does a length-R DFT and writes out[(j / Ns) Ns R + (j mod Ns) + r Ns].
//
// The density is real and so is the kernel K, which is even in each frequency:
// the potential's transform along x is conjugate-symmetric, so the passes keep
// kx <= M1 / 2 only and the last inverse x pass fills in the rest. That halves
// the lines of the y and z passes and their traffic.
//
// What bounds it: on the small boxes of a periodic cell the chain of stages
// (a barrier each; radix 8 makes 192 three stages and 32 two), on the doubled
// box of an isolated cell the index arithmetic and LDS passes ahead of HBM. So
// every quotient is a product with a float reciprocal, one table of the M
// roots serves all stages and both signs, and the lines of the y and z passes
// lie next to each other in LDS (eight lines are one 128-byte row: no bank
// conflict in any stage, and full lines of memory). The five passes of the
// 192^3 box of a 96^3 grid, before (complex, radix 4, divisions) and now:
// x 39 -> 23 us, y 60 -> 20, z with K 205 -> 58 (120 MB: 2.1 TB/s), inverse y
// 63 -> 20, inverse x 34 -> 27; a 36 x 40 x 27 cell's three launches by planes
// 36 -> 29 us.
struct FFTPlan {
  int M, nf;
  int f[12];
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// t / d for 0 <= t < 2^20 and inv = 1.0f / d: (t + 1/2) / d is at least
// 1 / (2 d) from an integer, the product's error below t / d 2^-22
__device__ __forceinline__ int quot(int t, float inv) { return (int)(((float)t + 0.5f) * inv); }

// o_s = sum_q v_q exp(sign 2 pi i q s / R) for R = 2, 3, 4, 5, 8
template <int R>
__device__ __forceinline__ void dft_small(double2* v, double sign);

template <>
__device__ __forceinline__ void dft_small<2>(double2* v, double) {
  const double2 a = v[0], b = v[1];
  v[0] = make_double2(a.x + b.x, a.y + b.y);
  v[1] = make_double2(a.x - b.x, a.y - b.y);
}

template <>
__device__ __forceinline__ void dft_small<4>(double2* v, double sign) {
  // omega = exp(sign i pi / 2) = sign * i
  const double2 a = v[0], b = v[1], c = v[2], d = v[3];
  const double2 s02 = make_double2(a.x + c.x, a.y + c.y), d02 = make_double2(a.x - c.x, a.y - c.y);
  const double2 s13 = make_double2(b.x + d.x, b.y + d.y), d13 = make_double2(b.x - d.x, b.y - d.y);
  // i * sign * d13
  const double2 r13 = make_double2(-sign * d13.y, sign * d13.x);
  v[0] = make_double2(s02.x + s13.x, s02.y + s13.y);
  v[1] = make_double2(d02.x + r13.x, d02.y + r13.y);
  v[2] = make_double2(s02.x - s13.x, s02.y - s13.y);
  v[3] = make_double2(d02.x - r13.x, d02.y - r13.y);
}

// two length-4 transforms (even and odd inputs) and a length-2 step with
// omega^s, omega = (1 + sign i) / sqrt(2)
template <>
__device__ __forceinline__ void dft_small<8>(double2* v, double sign) {
  double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
  dft_small<4>(e, sign);
  dft_small<4>(o, sign);
  const double h = 0.70710678118654752440;
  o[1] = make_double2(h * (o[1].x - sign * o[1].y), h * (sign * o[1].x + o[1].y));
  o[2] = make_double2(-sign * o[2].y, sign * o[2].x);
  o[3] = make_double2(-h * (o[3].x + sign * o[3].y), h * (sign * o[3].x - o[3].y));
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    v[s] = make_double2(e[s].x + o[s].x, e[s].y + o[s].y);
    v[s + 4] = make_double2(e[s].x - o[s].x, e[s].y - o[s].y);
  }
}

template <>
__device__ __forceinline__ void dft_small<3>(double2* v, double sign) {
  const double c1 = -0.5, s1 = sign * 0.86602540378443864676;  // exp(sign 2 pi i / 3)
  const double2 a = v[0], b = v[1], c = v[2];
  const double2 sbc = make_double2(b.x + c.x, b.y + c.y), dbc = make_double2(b.x - c.x, b.y - c.y);
  v[0] = make_double2(a.x + sbc.x, a.y + sbc.y);
  const double2 m = make_double2(a.x + c1 * sbc.x, a.y + c1 * sbc.y);
  // omega b + conj(omega) c = c1 (b + c) + i s1 (b - c)
  v[1] = make_double2(m.x - s1 * dbc.y, m.y + s1 * dbc.x);
  v[2] = make_double2(m.x + s1 * dbc.y, m.y - s1 * dbc.x);
}

template <>
__device__ __forceinline__ void dft_small<5>(double2* v, double sign) {
  const double cs[5] = {1.0, 0.30901699437494742410, -0.80901699437494742410, -0.80901699437494742410,
                        0.30901699437494742410};
  const double sn[5] = {0.0, 0.95105651629515357212, 0.58778525229247312917, -0.58778525229247312917,
                        -0.95105651629515357212};
  double2 o[5];
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const int e = (q * s) % 5;
      const double c = cs[e], sv = sign * sn[e];
      re += v[q].x * c - v[q].y * sv;
      im += v[q].x * sv + v[q].y * c;
    }
    o[s] = make_double2(re, im);
  }
#pragma unroll
  for (int s = 0; s < 5; ++s) v[s] = o[s];
}

// nl lines in LDS: element e of line l at e * se + l * sl (one of se, sl is 1;
// consecutive threads take the neighbours along it)
struct LineSet {
  int nl, se, sl;
};

// one stage; w: the M roots exp(2 pi i k / M), step = M / (Ns R)
template <int R>
__device__ __forceinline__ void stockham_stage(const double2* in, double2* out, const LineSet& ls, int M, int Ns,
                                               int step, double sign, const double2* w) {
  const int nb = M / R;
  const bool across = ls.sl == 1;
  const int d = across ? ls.nl : nb;
  const float inv_d = 1.0f / (float)d, inv_Ns = 1.0f / (float)Ns;
  for (int t = threadIdx.x; t < ls.nl * nb; t += blockDim.x) {
    const int q = quot(t, inv_d), rest = t - q * d;
    const int line = across ? rest : q, jj = across ? q : rest;
    const double2* li = in + line * ls.sl + jj * ls.se;
    const int jq = quot(jj, inv_Ns), jm = jj - jq * Ns;
    double2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = li[r * nb * ls.se];
    if (Ns > 1) {
      const int k = jm * step;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const double2 c = w[r * k];
        v[r] = cmul(v[r], make_double2(c.x, sign * c.y));
      }
    }
    dft_small<R>(v, sign);
    double2* lo = out + line * ls.sl + (jq * Ns * R + jm) * ls.se;
#pragma unroll
    for (int r = 0; r < R; ++r) lo[r * Ns * ls.se] = v[r];
  }
}

// the M roots exp(2 pi i k / M), by the workgroup's last wavefronts (all but
// the last `skip`): the first ones have the pass's loads to wait for
__device__ __forceinline__ void fft_roots(int M, double2* w, int skip = 0) {
  int k0 = (int)blockDim.x - 1 - (int)threadIdx.x - 64 * skip;
  if (k0 < 0) k0 += blockDim.x;
  for (int k = k0; k < M; k += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * (double)k / (double)M, &sn, &cs);
    w[k] = make_double2(cs, sn);
  }
}

// the plan's stages on the lines in LDS (in -> out alternating, a barrier
// after each); returns the buffer that holds the result
__device__ __forceinline__ double2* fft_lines_lds(const FFTPlan& plan, double2* in, double2* out,
                                                  const LineSet& ls, double sign, const double2* w) {
  const int M = plan.M;
  int Ns = 1, step = M;
  for (int f = 0; f < plan.nf; ++f) {
    const int R = plan.f[f];
    if (R == 8) stockham_stage<8>(in, out, ls, M, Ns, step /= 8, sign, w);
    else if (R == 4) stockham_stage<4>(in, out, ls, M, Ns, step /= 4, sign, w);
    else if (R == 2) stockham_stage<2>(in, out, ls, M, Ns, step /= 2, sign, w);
    else if (R == 3) stockham_stage<3>(in, out, ls, M, Ns, step /= 3, sign, w);
    else stockham_stage<5>(in, out, ls, M, Ns, step /= 5, sign, w);
    __syncthreads();
    Ns *= R;
    double2* t = in;
    in = out;
    out = t;
  }
  return in;
}

// The lines a pass transforms and the part of each it reads and writes: lines
// (i1, i2) with i1 < l1, i2 < l2 — (y, z) for the x axis, (x, z) for y, (x, y)
// for z — elements at or beyond n_in read as 0, elements at or beyond n_out
// not stored. ends (FFTEnds) says what else a pass does, so that it costs no
// launch of its own.
struct FFTLines {
  int l1, l2, n_in, n_out, ends;
  int B, nb1;  // lines per workgroup (of one i2) and workgroups per i2
};

// B lines of one pass (smem_raw: the dynamic LDS)
__device__ __forceinline__ void fft_axis_block(double2* data, int M1, int M2, int axis, int sign, const FFTPlan& plan,
                                               const double* rho, int n1, int n2, const double* K,
                                               const FFTLines& ln, int blk, unsigned char* smem_raw) {
  const int M = plan.M, B = ln.B;
  double2* buf0 = reinterpret_cast<double2*>(smem_raw);
  double2* buf1 = buf0 + B * M;
  double2* w = buf1 + B * M;
  const int i2 = blk / ln.nb1, i1 = (blk - i2 * ln.nb1) * B;
  const int nl = min(B, ln.l1 - i1);
  // element e of line l at base + l * gl + e * ge
  const size_t ge = axis == 0 ? 1 : (axis == 1 ? (size_t)M1 : (size_t)M1 * M2);
  const size_t gl = axis == 0 ? (size_t)M1 : 1;
  const size_t base = axis == 0 ? ((size_t)i2 * M2 + i1) * M1
                                : (axis == 1 ? (size_t)i2 * M1 * M2 + i1 : (size_t)i2 * M1 + i1);
  const LineSet ls{nl, axis == 0 ? 1 : B, axis == 0 ? M : 1};
  const int d = axis == 0 ? M : nl;
  const float inv_d = 1.0f / (float)d;
  const int total = nl * M;
  fft_roots(M, w);
  for (int i = threadIdx.x; i < total; i += blockDim.x) {
    const int q = quot(i, inv_d), rest = i - q * d;
    const int line = axis == 0 ? q : rest, e = axis == 0 ? rest : q;
    double2 v = make_double2(0.0, 0.0);
    if (ln.ends == kRho) {
      if (e < ln.n_in) v.x = rho[((size_t)i2 * n2 + i1 + line) * n1 + e];
    } else if (ln.ends == kConj && 2 * e > M) {
      v = data[base + line * gl + (M - e)];
      v.y = -v.y;
    } else if (e < ln.n_in) {
      v = data[base + line * gl + e * ge];
    }
    buf0[line * ls.sl + e * ls.se] = v;
  }
  // the kernel's values are in flight under the forward transform (a thread has
  // at most kKeep of them, but for lines beyond 2048)
  constexpr int kKeep = 4;
  double kv[kKeep];
  if (ln.ends == kKernel) {
#pragma unroll
    for (int u = 0; u < kKeep; ++u) {
      const int i = min((int)threadIdx.x + u * (int)blockDim.x, total - 1), e = quot(i, inv_d);
      kv[u] = K[base + (i - e * d) + e * ge];
    }
  }
  __syncthreads();
  double2* res = fft_lines_lds(plan, buf0, buf1, ls, (double)sign, w);
  if (ln.ends == kKernel) {
    auto times = [&](int i, double k, int e) {
      double2* r = res + (i - e * d) + e * B;
      *r = make_double2(r->x * k, r->y * k);
    };
#pragma unroll
    for (int u = 0; u < kKeep; ++u) {
      const int i = (int)threadIdx.x + u * (int)blockDim.x;
      if (i < total) times(i, kv[u], quot(i, inv_d));
    }
    for (int i = (int)threadIdx.x + kKeep * (int)blockDim.x; i < total; i += blockDim.x) {
      const int e = quot(i, inv_d);
      times(i, K[base + (i - e * d) + e * ge], e);
    }
    __syncthreads();
    res = fft_lines_lds(plan, res, res == buf0 ? buf1 : buf0, ls, -(double)sign, w);
  }
  for (int i = threadIdx.x; i < total; i += blockDim.x) {
    const int q = quot(i, inv_d), rest = i - q * d;
    const int line = axis == 0 ? q : rest, e = axis == 0 ? rest : q;
    if (e < ln.n_out) data[base + line * gl + e * ge] = res[line * ls.sl + e * ls.se];
  }
}

constexpr int kFFTThreads = 512;

__global__ __launch_bounds__(kFFTThreads) void k_fft_axis(double2* data, int M1, int M2, int axis, int sign,
                                                          FFTPlan plan, const double* rho, int n1, int n2,
                                                          const double* K, FFTLines ln) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  fft_axis_block(data, M1, M2, axis, sign, plan, rho, n1, n2, K, ln, (int)blockIdx.x, smem_raw);
}

// the same pass for the cells of a group (cell blockIdx.y)
__global__ __launch_bounds__(kFFTThreads) void k_fft_axis_group(const TailCell* __restrict__ tab, int M1, int M2,
                                                                int axis, int sign, FFTPlan plan, int n1, int n2,
                                                                FFTLines ln) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const TailCell& t = tab[blockIdx.y];
  fft_axis_block(t.fft, M1, M2, axis, sign, plan, t.rho, n1, n2, t.Kfft, ln, (int)blockIdx.x, smem_raw);
}

// the radix plan of a transform of length M (false: M has other prime
// factors): eights, with 2 x 8 as 4 x 4, then 4 or 2, threes and fives
static bool fft_plan(int M, FFTPlan* plan) {
  plan->M = M;
  plan->nf = 0;
  int rem = M, twos = 0;
  if (M < 1) return false;
  while (rem % 2 == 0) rem /= 2, ++twos;
  int n8 = twos / 3, left = twos - 3 * n8;
  if (left == 1 && n8 > 0) --n8, left = 4;
  for (int i = 0; i < n8 && plan->nf < 12; ++i) plan->f[plan->nf++] = 8;
  for (; left >= 2 && plan->nf < 12; left -= 2) plan->f[plan->nf++] = 4;
  if (left == 1 && plan->nf < 12) plan->f[plan->nf++] = 2;
  for (int r : {3, 5})
    while (rem % r == 0 && plan->nf < 12) {
      plan->f[plan->nf++] = r;
      rem /= r;
    }
  return rem == 1;
}

// lines, workgroups, threads and LDS of a pass over ncells boxes: up to 2048
// points a workgroup (eight lines of 192), fewer until min_wg workgroups share
// the pass; threads for a radix-4 butterfly each
struct FFTShape {
  FFTLines ln;
  unsigned grid;
  int threads;
  size_t lds;
};
static FFTShape fft_shape(int M, int l1, int l2, int n_in, int n_out, int ends, int ncells, int min_wg) {
  int B = 1;
  while (2 * B * M <= 2048 && B < l1) B *= 2;
  auto groups = [&](int b) { return (long)((l1 + b - 1) / b) * l2; };
  while (B > 1 && groups(B) * ncells < min_wg) B /= 2;
  FFTShape f;
  f.ln = FFTLines{l1, l2, n_in, n_out, ends, B, (l1 + B - 1) / B};
  f.grid = (unsigned)groups(B);
  f.threads = min(kFFTThreads, max(64, (B * M / 4 + 63) / 64 * 64));
  f.lds = ((size_t)2 * B * M + (size_t)M) * sizeof(double2);
  return f;
}

hipError_t launch_fft_lines_group(const TailCell* tab, int ncells, int M1, int M2, int M3, int axis, int sign,
                                  int ends, int n1, int n2, int l1, int l2, int n_in, int n_out, hipStream_t s) {
  FFTPlan plan;
  if (!fft_plan(axis == 0 ? M1 : (axis == 1 ? M2 : M3), &plan)) return hipErrorInvalidValue;
  if ((ends == kKernel && axis != 2) || ((ends == kRho || ends == kConj) && axis != 0)) return hipErrorInvalidValue;
  if (l1 <= 0 || l2 <= 0 || ncells <= 0) return hipSuccess;
  // a workgroup per compute unit over all cells (two cells of 16^3 on four
  // workgroups took 14 us a pass)
  const FFTShape f = fft_shape(plan.M, l1, l2, n_in, n_out, ends, ncells, 256);
  hipLaunchKernelGGL(k_fft_axis_group, dim3(f.grid, ncells), dim3(f.threads), f.lds, s, tab, M1, M2, axis, sign,
                     plan, n1, n2, f.ln);
  return hipGetLastError();
}

hipError_t launch_fft_lines(double2* data, int M1, int M2, int M3, int axis, int sign, hipStream_t s, int ends,
                            const double* rho, int n1, int n2, const double* K, int l1, int l2, int n_in,
                            int n_out) {
  FFTPlan plan;
  if (!fft_plan(axis == 0 ? M1 : (axis == 1 ? M2 : M3), &plan)) return hipErrorInvalidValue;
  if ((ends == kKernel && (axis != 2 || !K)) || (ends == kRho && (axis != 0 || !rho)) || (ends == kConj && axis != 0))
    return hipErrorInvalidValue;
  if (l1 <= 0 || l2 <= 0) return hipSuccess;
  const FFTShape f = fft_shape(plan.M, l1, l2, n_in, n_out, ends, 1, 64);
  hipLaunchKernelGGL(k_fft_axis, dim3(f.grid), dim3(f.threads), f.lds, s, data, M1, M2, axis, sign, plan, rho, n1,
                     n2, K, f.ln);
  return hipGetLastError();
}

hipError_t launch_fft_axis(double2* data, int M1, int M2, int M3, int axis, int sign, hipStream_t s) {
  const int l1 = axis == 0 ? M2 : M1, l2 = axis == 2 ? M2 : M3;
  const int M = axis == 0 ? M1 : (axis == 1 ? M2 : M3);
  return launch_fft_lines(data, M1, M2, M3, axis, sign, s, kPlain, nullptr, 0, 0, nullptr, l1, l2, M, M);
}

// ---------------------------------------------------------------- LDA + V
// Perdew-Zunger 1981, spin-unpolarised; r_s >= 1 uses the Pade form in
// sqrt(r_s), r_s < 1 the high-density logarithmic form; rho < 1e-30 -> 0.
// exchange_too = 0 leaves out the LDA exchange potential (the BJ / TB09
// exchange replaces it); e is always the full LDA energy density
__device__ void pz81(double rho, int exchange_too, double* v, double* e) {
  if (!(rho >= 1e-30)) {
    *v = 0.0;
    *e = 0.0;
    return;
  }
  const double third = 1.0 / 3.0;
  const double pi = 3.14159265358979323846;
  const double rs = cbrt(3.0 / (4.0 * pi * rho));
  const double vx = -cbrt(3.0 * rho / pi);
  const double ex = 0.75 * vx;
  double ec, vc;
  if (rs >= 1.0) {
    const double g = -0.1423, b1 = 1.0529, b2 = 0.3334;
    const double sq = sqrt(rs);
    const double den = 1.0 + b1 * sq + b2 * rs;
    ec = g / den;
    vc = ec * (1.0 + 7.0 / 6.0 * b1 * sq + 4.0 / 3.0 * b2 * rs) / den;
  } else {
    const double A = 0.0311, B = -0.048, C = 0.0020, D = -0.0116;
    const double l = log(rs);
    ec = A * l + B + C * rs * l + D * rs;
    vc = A * l + (B - A * third) + 2.0 * third * C * rs * l + (2.0 * D - C) * third * rs;
  }
  *v = exchange_too ? vx + vc : vc;
  *e = ex + ec;
}

// xc: 0 none, 1 PZ81, 2 and 3 the exchange in vx_mgga plus PZ81 correlation
__device__ __forceinline__ void xc_value(double vh, double rho, double Vloc, int xc, double vx_mgga, double* Vd,
                                         float* Vf, double* vh_out, double* exc, size_t p) {
  double vxc = 0.0, e = 0.0;
  if (xc) {
    pz81(rho, xc == 1, &vxc, &e);
    if (xc >= 2) vxc += vx_mgga;
  }
  const double v = Vloc + vh + vxc;
  Vd[p] = v;
  Vf[p] = (float)v;
  vh_out[p] = vh;
  exc[p] = e;
}

__device__ __forceinline__ void xc_point(const double2* data, int n1, int n2, int M1, int M2, double vh_scale,
                                         const double* rho, const double* Vloc, int hartree, int xc,
                                         const double* vx_mgga, double* Vd, float* Vf, double* vh_out,
                                         double* exc, size_t p) {
  const int x = (int)(p % n1);
  const int y = (int)((p / n1) % n2);
  const int z = (int)(p / ((size_t)n1 * n2));
  double vh = 0.0;
  if (hartree) vh = data[((size_t)z * M2 + y) * M1 + x].x * vh_scale;
  xc_value(vh, rho[p], Vloc[p], xc, xc >= 2 ? vx_mgga[p] : 0.0, Vd, Vf, vh_out, exc, p);
}

// ---------------------------------------------------------------- Poisson by planes
// For a periodic box whose xy plane fits a workgroup the Poisson solve is
// three launches: (1) per z plane, the density summed over its chunks and the
// forward transforms along x and y in LDS; (2) the z lines, forward, kernel,
// inverse (k_fft_axis); (3) per plane the inverse transforms along y and x and
// the potential. Each line is transformed as in the pass-by-pass form (which
// isolated boxes and larger planes use), so the bits of the solve are the same;
// that form's reduction, five passes and assembly are seven launches of 4 to
// 7 us each, half of a small cell's step. The plane stays [y][x] in LDS for
// both directions (the stages take the stride), and only kx <= n1 / 2 goes
// through the y transforms and memory. What is left is latency: loads go out
// before they are needed and the roots are formed by wavefronts that wait for
// none (16^3, one chunk of orbitals: 21 -> 15 us for the three launches).
struct PlanePlan {
  int n1, n2, n3;
  FFTPlan x, y;
};
constexpr int kPlaneThreads = 1024;  // every launch's

bool poisson_planes(int periodic, int hartree, int n1, int n2) {
  return periodic && hartree && n1 * n2 <= kPlaneMax;
}

// the roots of both lengths (one table where they are equal)
__device__ __forceinline__ const double2* plane_roots(const PlanePlan& pl, double2* wx) {
  fft_roots(pl.n1, wx);
  if (pl.n1 == pl.n2) return wx;
  fft_roots(pl.n2, wx + pl.n1, 1);
  return wx + pl.n1;
}

__device__ __forceinline__ void poisson_forward_plane(const TailCell& t, const PlanePlan& pl, int z,
                                                      unsigned char* smem_raw) {
  const int P = pl.n1 * pl.n2;
  const size_t N = (size_t)P * pl.n3;
  double2* a = reinterpret_cast<double2*>(smem_raw);
  double2* b = a + P;
  double2* wx = b + P;
  const double2* wy = plane_roots(pl, wx);
  double* rho = t.rho + (size_t)z * P;
  if (t.nchunks == 1) {
    for (int p = threadIdx.x; p < P; p += blockDim.x) a[p] = make_double2(rho[p], 0.0);
  } else {
    // slices of the workgroup sum chunks j, j + nsl, ... in order, then the
    // slices add up in order
    const int nsl = max(1, (int)blockDim.x / P);
    double* red = reinterpret_cast<double*>(wx + pl.n1 + pl.n2);  // [nsl][P] (nsl > 1: at most blockDim.x)
    const double* part = t.rho_part + (size_t)z * P;
    for (int i = threadIdx.x; i < nsl * P; i += blockDim.x) {
      const int j = i / P, p = i - j * P;
      double acc = 0.0;
      for (int c = j; c < t.nchunks; c += kRhoPipe * nsl) {
        double v[kRhoPipe];
#pragma unroll
        for (int u = 0; u < kRhoPipe; ++u) v[u] = part[(size_t)min(c + u * nsl, t.nchunks - 1) * N + p];
#pragma unroll
        for (int u = 0; u < kRhoPipe; ++u) acc += c + u * nsl < t.nchunks ? v[u] : 0.0;
      }
      if (nsl == 1) {
        rho[p] = acc;
        a[p] = make_double2(acc, 0.0);
      } else {
        red[i] = acc;
      }
    }
    if (nsl > 1) {
      __syncthreads();
      for (int p = threadIdx.x; p < P; p += blockDim.x) {
        double acc = red[p];
        for (int j = 1; j < nsl; ++j) acc += red[j * P + p];
        rho[p] = acc;
        a[p] = make_double2(acc, 0.0);
      }
    }
  }
  __syncthreads();
  const int H = pl.n1 / 2 + 1;
  double2* r = fft_lines_lds(pl.x, a, b, LineSet{pl.n2, 1, pl.n1}, -1.0, wx);
  r = fft_lines_lds(pl.y, r, r == a ? b : a, LineSet{H, pl.n1, 1}, -1.0, wy);
  double2* out = t.fft + (size_t)z * P;
  const float inv = 1.0f / (float)H;
  for (int i = threadIdx.x; i < H * pl.n2; i += blockDim.x) {
    const int y = quot(i, inv), p = y * pl.n1 + i - y * H;
    out[p] = r[p];
  }
}

__device__ __forceinline__ void poisson_inverse_plane(const TailCell& t, const PlanePlan& pl, int xc,
                                                      const double* vx_mgga, int z, unsigned char* smem_raw) {
  const int P = pl.n1 * pl.n2;
  double2* a = reinterpret_cast<double2*>(smem_raw);
  double2* b = a + P;
  double2* wx = b + P;
  const double2* wy = plane_roots(pl, wx);
  const double2* in = t.fft + (size_t)z * P;
  const int H = pl.n1 / 2 + 1;
  const float inv = 1.0f / (float)H;
  for (int i = threadIdx.x; i < H * pl.n2; i += blockDim.x) {
    const int y = quot(i, inv), p = y * pl.n1 + i - y * H;
    a[p] = in[p];
  }
  // what the potential needs besides is in flight under the transforms
  constexpr int kKeep = kPlaneMax / kPlaneThreads;
  double rho[kKeep], vloc[kKeep], vx[kKeep];
#pragma unroll
  for (int u = 0; u < kKeep; ++u) {
    const size_t p = (size_t)z * P + min((int)threadIdx.x + u * kPlaneThreads, P - 1);
    rho[u] = t.rho[p];
    vloc[u] = t.Vloc[p];
    vx[u] = xc >= 2 ? vx_mgga[p] : 0.0;
  }
  __syncthreads();
  double2* r = fft_lines_lds(pl.y, a, b, LineSet{H, pl.n1, 1}, +1.0, wy);
  // kx > n1 / 2 from its conjugate
  const int C = pl.n1 - H;
  const float invC = 1.0f / (float)C;
  for (int i = threadIdx.x; i < C * pl.n2; i += blockDim.x) {
    const int y = quot(i, invC), x = H + i - y * C;
    const double2 v = r[y * pl.n1 + pl.n1 - x];
    r[y * pl.n1 + x] = make_double2(v.x, -v.y);
  }
  __syncthreads();
  r = fft_lines_lds(pl.x, r, r == a ? b : a, LineSet{pl.n2, 1, pl.n1}, +1.0, wx);
#pragma unroll
  for (int u = 0; u < kKeep; ++u) {
    const int i = (int)threadIdx.x + u * kPlaneThreads;
    if (i < P)
      xc_value(r[i].x * t.vh_scale, rho[u], vloc[u], xc, vx[u], t.Vd, t.Vf, t.vh, t.exc, (size_t)z * P + i);
  }
}

__global__ __launch_bounds__(kPlaneThreads) void k_poisson_forward(TailCell t, PlanePlan pl) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  poisson_forward_plane(t, pl, (int)blockIdx.x, smem_raw);
}
__global__ __launch_bounds__(kPlaneThreads) void k_poisson_inverse(TailCell t, PlanePlan pl, int xc,
                                                                   const double* vx_mgga) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  poisson_inverse_plane(t, pl, xc, vx_mgga, (int)blockIdx.x, smem_raw);
}
// the same for the cells of a group (cell blockIdx.y; LDA or no xc)
__global__ __launch_bounds__(kPlaneThreads) void k_poisson_forward_group(const TailCell* __restrict__ tab,
                                                                         PlanePlan pl) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  poisson_forward_plane(tab[blockIdx.y], pl, (int)blockIdx.x, smem_raw);
}
__global__ __launch_bounds__(kPlaneThreads) void k_poisson_inverse_group(const TailCell* __restrict__ tab,
                                                                         PlanePlan pl, int xc) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  poisson_inverse_plane(tab[blockIdx.y], pl, xc, nullptr, (int)blockIdx.x, smem_raw);
}

static bool plane_plan(int n1, int n2, int n3, PlanePlan* pl, size_t* lds, int* threads) {
  pl->n1 = n1;
  pl->n2 = n2;
  pl->n3 = n3;
  *lds = ((size_t)2 * n1 * n2 + n1 + n2) * sizeof(double2) + kPlaneThreads * sizeof(double);
  *threads = kPlaneThreads;
  return n1 * n2 <= kPlaneMax && fft_plan(n1, &pl->x) && fft_plan(n2, &pl->y);
}

hipError_t launch_poisson_forward(const TailCell& t, int n1, int n2, int n3, hipStream_t s) {
  PlanePlan pl;
  size_t lds;
  int th;
  if (!plane_plan(n1, n2, n3, &pl, &lds, &th)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_poisson_forward, dim3(n3), dim3(th), lds, s, t, pl);
  return hipGetLastError();
}
hipError_t launch_poisson_inverse(const TailCell& t, int n1, int n2, int n3, int xc, const double* vx_mgga,
                                  hipStream_t s) {
  PlanePlan pl;
  size_t lds;
  int th;
  if (!plane_plan(n1, n2, n3, &pl, &lds, &th)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_poisson_inverse, dim3(n3), dim3(th), lds, s, t, pl, xc, vx_mgga);
  return hipGetLastError();
}
hipError_t launch_poisson_forward_group(const TailCell* tab, int ncells, int n1, int n2, int n3, hipStream_t s) {
  PlanePlan pl;
  size_t lds;
  int th;
  if (!plane_plan(n1, n2, n3, &pl, &lds, &th)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_poisson_forward_group, dim3(n3, ncells), dim3(th), lds, s, tab, pl);
  return hipGetLastError();
}
hipError_t launch_poisson_inverse_group(const TailCell* tab, int ncells, int n1, int n2, int n3, int xc,
                                        hipStream_t s) {
  PlanePlan pl;
  size_t lds;
  int th;
  if (xc >= 2 || !plane_plan(n1, n2, n3, &pl, &lds, &th)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_poisson_inverse_group, dim3(n3, ncells), dim3(th), lds, s, tab, pl, xc);
  return hipGetLastError();
}

__global__ void k_xc_assemble(const double2* data, int n1, int n2, int n3, int M1, int M2,
                              double vh_scale, const double* rho, const double* Vloc, int hartree,
                              int xc, const double* vx_mgga, double* Vd, float* Vf, double* vh_out,
                              double* exc) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t N = (size_t)n1 * n2 * n3;
  if (p >= N) return;
  xc_point(data, n1, n2, M1, M2, vh_scale, rho, Vloc, hartree, xc, vx_mgga, Vd, Vf, vh_out, exc, p);
}

// the same for the cells of a group (cell blockIdx.y; LDA or no xc)
__global__ void k_xc_group(const TailCell* __restrict__ tab, int n1, int n2, int n3, int M1, int M2, int hartree,
                           int xc) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t N = (size_t)n1 * n2 * n3;
  if (p >= N) return;
  const TailCell& t = tab[blockIdx.y];
  xc_point(t.fft, n1, n2, M1, M2, t.vh_scale, t.rho, t.Vloc, hartree, xc, nullptr, t.Vd, t.Vf, t.vh, t.exc, p);
}

hipError_t launch_xc_group(const TailCell* tab, int ncells, int n1, int n2, int n3, int M1, int M2, int hartree,
                           int xc, hipStream_t s) {
  if (xc >= 2) return hipErrorInvalidValue;
  const size_t N = (size_t)n1 * n2 * n3;
  hipLaunchKernelGGL(k_xc_group, dim3((unsigned)((N + 255) / 256), ncells), dim3(256), 0, s, tab, n1, n2, n3, M1,
                     M2, hartree, xc);
  return hipGetLastError();
}

hipError_t launch_xc_assemble(const double2* data, int n1, int n2, int n3, int M1, int M2, int M3,
                              double vh_scale, const double* rho, const double* Vloc, int hartree,
                              int xc, const double* vx_mgga, double* Vd, float* Vf, double* vh, double* exc,
                              hipStream_t s) {
  (void)M3;
  const size_t N = (size_t)n1 * n2 * n3;
  hipLaunchKernelGGL(k_xc_assemble, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, data, n1, n2,
                     n3, M1, M2, vh_scale, rho, Vloc, hartree, xc, vx_mgga, Vd, Vf, vh, exc);
  return hipGetLastError();
}

// ---------------------------------------------------------------- grid sums
// out[0] = 1/2 h^3 sum rho V_H, out[1] = h^3 sum rho eps_xc,
// out[2..4] = -h^3 sum (r - centre)(rho - rho0), out[5] = h^3 sum rho.
__global__ __launch_bounds__(1024) void k_grid_sums(const double* rho, const double* rho0,
                                                    const double* vh, const double* exc, Geometry g,
                                                    double* out) {
  __shared__ double red[1024][6];
  const int t = threadIdx.x;
  const size_t N = (size_t)g.n1 * g.n2 * g.n3;
  double s[6] = {0, 0, 0, 0, 0, 0};
  for (size_t p = t; p < N; p += blockDim.x) {
    const int x = (int)(p % g.n1);
    const int y = (int)((p / g.n1) % g.n2);
    const int z = (int)(p / ((size_t)g.n1 * g.n2));
    const double r = rho[p];
    const double dr = r - rho0[p];
    s[0] += r * vh[p];
    s[1] += r * exc[p];
    s[2] += (x - 0.5 * (g.n1 - 1)) * g.h1 * dr;
    s[3] += (y - 0.5 * (g.n2 - 1)) * g.h2 * dr;
    s[4] += (z - 0.5 * (g.n3 - 1)) * g.h3 * dr;
    s[5] += r;
  }
  for (int i = 0; i < 6; ++i) red[t][i] = s[i];
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (t < w)
      for (int i = 0; i < 6; ++i) red[t][i] += red[t + w][i];
    __syncthreads();
  }
  if (t == 0) {
    const double dV = g.h1 * g.h2 * g.h3;
    out[0] = 0.5 * dV * red[0][0];
    out[1] = dV * red[0][1];
    out[2] = -dV * red[0][2];
    out[3] = -dV * red[0][3];
    out[4] = -dV * red[0][4];
    out[5] = dV * red[0][5];
  }
}

hipError_t launch_grid_sums(const double* rho, const double* rho0, const double* vh,
                            const double* exc, Geometry g, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_grid_sums, dim3(1), dim3(1024), 0, s, rho, rho0, vh, exc, g, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- conversions
template <typename T>
__global__ void k_convert_in(const double2* src, typename Vec2<T>::type* dst, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 v = src[i];
  typename Vec2<T>::type o;
  o.x = (T)v.x;
  o.y = (T)v.y;
  dst[i] = o;
}
template <typename T>
__global__ void k_convert_out(const typename Vec2<T>::type* src, double2* dst, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const auto v = src[i];
  dst[i] = make_double2((double)v.x, (double)v.y);
}
template <typename T>
hipError_t launch_convert_in(const double2* src, typename Vec2<T>::type* dst, size_t n, hipStream_t s) {
  hipLaunchKernelGGL((k_convert_in<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_convert_out(const typename Vec2<T>::type* src, double2* dst, size_t n, hipStream_t s) {
  hipLaunchKernelGGL((k_convert_out<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}
template hipError_t launch_convert_in<double>(const double2*, double2*, size_t, hipStream_t);
template hipError_t launch_convert_in<float>(const double2*, float2*, size_t, hipStream_t);
template hipError_t launch_convert_out<double>(const double2*, double2*, size_t, hipStream_t);
template hipError_t launch_convert_out<float>(const float2*, double2*, size_t, hipStream_t);

// w <- exp(-i F0 r_axis) w with r from the box centre (isolated kick, Sec. 3.1)
template <typename T>
__global__ void k_kick(typename Vec2<T>::type* w, Geometry g, double F0, int axis, size_t total) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const size_t N = (size_t)g.n1 * g.n2 * g.n3;
  const size_t p = i % N;
  int c;
  double h;
  int n;
  if (axis == 0) {
    c = (int)(p % g.n1);
    h = g.h1;
    n = g.n1;
  } else if (axis == 1) {
    c = (int)((p / g.n1) % g.n2);
    h = g.h2;
    n = g.n2;
  } else {
    c = (int)(p / ((size_t)g.n1 * g.n2));
    h = g.h3;
    n = g.n3;
  }
  const double r = (c - 0.5 * (n - 1)) * h;
  double sn, cs;
  sincos(-F0 * r, &sn, &cs);
  auto v = w[i];
  const double re = (double)v.x, im = (double)v.y;
  v.x = (T)(re * cs - im * sn);
  v.y = (T)(re * sn + im * cs);
  w[i] = v;
}
template <typename T>
hipError_t launch_kick(typename Vec2<T>::type* w, Geometry g, double F0, int axis, size_t n_orb_tot,
                       hipStream_t s) {
  const size_t total = n_orb_tot * (size_t)g.n1 * g.n2 * g.n3;
  hipLaunchKernelGGL((k_kick<T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, w, g, F0,
                     axis, total);
  return hipGetLastError();
}
template hipError_t launch_kick<double>(double2*, Geometry, double, int, size_t, hipStream_t);
template hipError_t launch_kick<float>(float2*, Geometry, double, int, size_t, hipStream_t);

__global__ void k_real_part(const double2* src, double* dst, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i].x;
}
hipError_t launch_real_part(const double2* src, double* dst, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_real_part, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}

__global__ void k_fill(double* p, double v, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
hipError_t launch_fill(double* p, double v, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

// dst = src, 8 bytes per thread (both 8-byte aligned, bytes a multiple of 8)
__global__ void k_copy8(const double* __restrict__ src, double* __restrict__ dst, size_t n8) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n8) dst[i] = src[i];
}
hipError_t launch_copy8(const void* src, void* dst, size_t bytes, hipStream_t s) {
  const size_t n8 = bytes / 8;
  if (n8 == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy8, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s,
                     static_cast<const double*>(src), static_cast<double*>(dst), n8);
  return hipGetLastError();
}

// predictor-corrector: V = (V_n + V_pred) / 2 in FP64 and its stage-precision copy
__global__ void k_mid_potential(const double* __restrict__ Vn, double* __restrict__ Vd, float* __restrict__ Vf,
                                size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double v = 0.5 * (Vn[i] + Vd[i]);
  Vd[i] = v;
  Vf[i] = (float)v;
}
hipError_t launch_mid_potential(const double* Vn, double* Vd, float* Vf, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_mid_potential, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Vn, Vd, Vf, n);
  return hipGetLastError();
}

__global__ void k_set_int(int* p, int v) { *p = v; }
hipError_t launch_set_int(int* p, int v, hipStream_t s) {
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, s, p, v);
  return hipGetLastError();
}

}  // namespace td
