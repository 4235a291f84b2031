// Orthonormalisation of the orbitals of every k-point (Gram-Schmidt in
// orbital order, as Cholesky-QR): S_k[i][j] = h^3 sum_r w_i(r) conj(w_j(r))
// formed on the device in FP64 (fixed-order reductions), S_k = L L^H factored
// and inverted on the device, and w <- L^{-1} w applied there too. Used by the
// ground-state preparation that precedes the real-time run (Sec. 2.1).
#include "internal.h"

namespace td {

typedef double d4_t __attribute__((ext_vector_type(4)));

// Overlaps on the matrix cores: for a pair of 16-orbital tiles (ti >= tj) of a
// k-point and a chunk of grid points, the 16 x 16 block
//   S_re = sum_p ar br^T + ai bi^T,  S_im = sum_p ai br^T - ar bi^T
// (a, b: the tiles' orbitals) by v_mfma_f64_16x16x4f64, whose lane l takes
// A[l % 16][l / 16] and B[l / 16][l % 16] and leaves D[l / 16 + 4 r][l % 16]: a
// lane loads four consecutive points of one orbital and they serve as the k
// index of four products. part[..][512]: the chunk's block, real then
// imaginary. A workgroup per orbital pair read every orbital n_orb times
// (51 us for 64 k-points of 16 orbitals at 16^3); this reads each once per tile
// pair, 5 us.
template <typename T>
__global__ __launch_bounds__(256) void k_gram(const typename Vec2<T>::type* __restrict__ w, int n_orb, int N,
                                              int chunk, int nchunks, int ntiles, double* __restrict__ part) {
  __shared__ double red[4][8][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int b = blockIdx.x;
  const int ch = b % nchunks;
  b /= nchunks;
  const int k = b / ntiles;
  int pr = b - k * ntiles, ti = 0;
  while (pr > ti) {
    pr -= ti + 1;
    ++ti;
  }
  const int tj = pr;
  const int row = lane & 15, q = lane >> 4;
  const int oa = 16 * ti + row, ob = 16 * tj + row;
  const auto* wa = w + ((size_t)k * n_orb + min(oa, n_orb - 1)) * N;
  const auto* wb = w + ((size_t)k * n_orb + min(ob, n_orb - 1)) * N;
  const int p0 = ch * chunk, p1 = min(N, p0 + chunk);
  d4_t re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
  constexpr int kAhead = 2;  // groups of 16 points whose loads are issued together
  for (int pb = p0 + 16 * wave; pb < p1; pb += 64 * kAhead) {
    typename Vec2<T>::type va[kAhead][4], vb[kAhead][4];
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p = min(pb + 64 * u + 4 * q + e, p1 - 1);
        va[u][e] = wa[p];
        vb[u][e] = wb[p];
      }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = pb + 64 * u + 4 * q + e < p1;
        const double ar = in && oa < n_orb ? (double)va[u][e].x : 0.0, ai = in && oa < n_orb ? (double)va[u][e].y : 0.0;
        const double br = in && ob < n_orb ? (double)vb[u][e].x : 0.0, bi = in && ob < n_orb ? (double)vb[u][e].y : 0.0;
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, bi, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(-ar, bi, im, 0, 0, 0);
      }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    red[wave][r][lane] = re[r];
    red[wave][4 + r][lane] = im[r];
  }
  __syncthreads();
  double* out = part + (size_t)blockIdx.x * 512;
  for (int i = threadIdx.x; i < 512; i += 256) {
    const int c = i >> 6, l = i & 63;
    const double v = red[0][c][l] + red[1][c][l] + red[2][c][l] + red[3][c][l];
    out[(c >> 2) * 256 + ((l >> 4) + 4 * (c & 3)) * 16 + (l & 15)] = v;
  }
}

// the overlap of orbitals i >= j of a k-point: its tile's chunks in order
__device__ __forceinline__ double2 gram_entry(const double* __restrict__ part, int k, int ntiles, int nchunks,
                                              double dV, int i, int j) {
  const int ti = i >> 4, tj = j >> 4;
  const double* p = part + ((size_t)k * ntiles + ti * (ti + 1) / 2 + tj) * nchunks * 512 + (i & 15) * 16 + (j & 15);
  double re = 0.0, im = 0.0;
  constexpr int kAhead = 8;  // chunks whose loads are issued together
  for (int c0 = 0; c0 < nchunks; c0 += kAhead) {
    double vr[kAhead], vi[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const size_t at = (size_t)min(c0 + u, nchunks - 1) * 512;
      vr[u] = p[at];
      vi[u] = p[at + 256];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      re += c0 + u < nchunks ? vr[u] : 0.0;
      im += c0 + u < nchunks ? vi[u] : 0.0;
    }
  }
  return make_double2(dV * re, dV * im);
}

// S[k][i][j], i >= j
__global__ __launch_bounds__(256) void k_gram_reduce(const double* __restrict__ part, int n, int ntiles, int nchunks,
                                                     double dV, double2* __restrict__ S) {
  const int k = blockIdx.y, e = blockIdx.x * 256 + threadIdx.x;
  if (e >= n * n) return;
  const int i = e / n, j = e - i * n;
  if (i >= j) S[(size_t)k * n * n + e] = gram_entry(part, k, ntiles, nchunks, dV, i, j);
}

__device__ __forceinline__ double lane_read(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Up to 32 orbitals: the chunks' sums, the Cholesky factor and its inverse of
// one k-point per workgroup. One wavefront factors with a row per lane in
// registers (values of other rows by lane reads) and inverts with a column per
// lane; through memory, column by column, it took 38 us for 16 orbitals, this 8.
// Mt[k][c][i] = (L^{-1})_ic.
template <int NB>
__global__ __launch_bounds__(256) void k_chol_small(const double* __restrict__ part, int n, int ntiles, int nchunks,
                                                    double dV, double2* __restrict__ Mt, int* __restrict__ bad) {
  __shared__ double2 A[NB][NB + 1];
  const int k = blockIdx.x, tid = threadIdx.x;
  for (int e = tid; e < NB * NB; e += 256) {
    const int i = e / NB, j = e % NB;
    double2 v = make_double2(i == j ? 1.0 : 0.0, 0.0);
    if (i < n && j <= i) v = gram_entry(part, k, ntiles, nchunks, dV, i, j);
    A[i][j] = v;
  }
  __syncthreads();
  if (tid >= 64) return;
  const int r = tid % NB;
  double ar[NB], ai[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    ar[c] = A[r][c].x;
    ai[c] = A[r][c].y;
  }
  bool good = true;
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    double d = lane_read(ar[c], c);
    if (!(d > 0.0)) {
      good = false;
      d = 1.0;
    }
    const double piv = sqrt(d);
    ar[c] = r == c ? piv : ar[c] / piv;
    ai[c] = r == c ? 0.0 : ai[c] / piv;
    // row r less L_rc times row k's conj(L_kc) (of use where r >= k)
#pragma unroll
    for (int q = c + 1; q < NB; ++q) {
      const double lr = lane_read(ar[c], q), li = lane_read(ai[c], q);
      ar[q] -= ar[c] * lr + ai[c] * li;
      ai[q] -= ai[c] * lr - ar[c] * li;
      // keeps the next lane reads (scalar registers) behind this update
      asm volatile("" : "+v"(ar[c]), "+v"(ai[c]), "+v"(ar[q]), "+v"(ai[q]));
    }
  }
  if (!good && tid == 0) atomicOr(bad, 1);
  // opaque: the inversion would otherwise keep the factorisation's lane reads
#pragma unroll
  for (int c = 0; c < NB; ++c) asm volatile("" : "+v"(ar[c]), "+v"(ai[c]));
  double mr[NB], mi[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    double br = i == r ? 1.0 : 0.0, bi = 0.0;
#pragma unroll
    for (int q = 0; q < i; ++q) {
      const double lr = lane_read(ar[q], i), li = lane_read(ai[q], i);
      br -= lr * mr[q] - li * mi[q];
      bi -= lr * mi[q] + li * mr[q];
      asm volatile("" : "+v"(br), "+v"(bi), "+v"(ar[q + 1]), "+v"(ai[q + 1]));
    }
    const double d = lane_read(ar[i], i);
    mr[i] = br / d;
    mi[i] = bi / d;
  }
  if (tid < n) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (i < n) Mt[((size_t)k * n + tid) * n + i] = make_double2(mr[i], mi[i]);
  }
}

// Per k-point (one workgroup each): the Cholesky factor S = L L^H of the
// Hermitian positive overlap matrix (left-looking, column by column; L
// overwrites the lower triangle of S) and its inverse M = L^{-1} (lower
// triangular, stored by columns; the columns are independent, one thread each).
// A pivot that is not positive sets *bad (the orbitals became linearly
// dependent). More than 32 orbitals; fewer take k_chol_small.
__global__ __launch_bounds__(256) void k_chol_inverse(double2* __restrict__ S, double2* __restrict__ M, int n,
                                                      int* __restrict__ bad) {
  __shared__ double piv;
  const int k = blockIdx.x;
  double2* L = S + (size_t)k * n * n;
  double2* Mk = M + (size_t)k * n * n;
  const int t = threadIdx.x, nt = blockDim.x;
  for (int j = 0; j < n; ++j) {
    // s_ij = S_ij - sum_{q<j} L_iq conj(L_jq), for i >= j
    for (int i = j + t; i < n; i += nt) {
      double sr = L[(size_t)i * n + j].x, si = L[(size_t)i * n + j].y;
      for (int q = 0; q < j; ++q) {
        const double2 a = L[(size_t)i * n + q], b = L[(size_t)j * n + q];
        sr -= a.x * b.x + a.y * b.y;
        si -= a.y * b.x - a.x * b.y;
      }
      L[(size_t)i * n + j] = make_double2(sr, si);
    }
    __syncthreads();
    if (t == 0) {
      const double d = L[(size_t)j * n + j].x;
      if (!(d > 0.0)) atomicOr(bad, 1);
      piv = d > 0.0 ? sqrt(d) : 1.0;
      L[(size_t)j * n + j] = make_double2(piv, 0.0);
    }
    __syncthreads();
    for (int i = j + 1 + t; i < n; i += nt) {
      const double2 v = L[(size_t)i * n + j];
      L[(size_t)i * n + j] = make_double2(v.x / piv, v.y / piv);
    }
    __syncthreads();
  }
  // M = L^{-1}: column c by forward substitution, M_ic = (delta_ic - sum_{q=c}^{i-1} L_iq M_qc) / L_ii
  for (int c = t; c < n; c += nt) {
    for (int i = 0; i < c; ++i) Mk[(size_t)c * n + i] = make_double2(0.0, 0.0);
    for (int i = c; i < n; ++i) {
      double br = (i == c) ? 1.0 : 0.0, bi = 0.0;
      for (int q = c; q < i; ++q) {
        const double2 l = L[(size_t)i * n + q], m = Mk[(size_t)c * n + q];
        br -= l.x * m.x - l.y * m.y;
        bi -= l.x * m.y + l.y * m.x;
      }
      const double d = L[(size_t)i * n + i].x;
      Mk[(size_t)c * n + i] = make_double2(br / d, bi / d);
    }
  }
}

// w[k][i][p] <- sum_{j <= i} M[k][i][j] w[k][j][p] in place on the matrix cores:
// 16 x 16 blocks of M times 16 orbitals by 16 points, v_mfma_f64_16x16x4f64 with
// the orbital j as its k index. A wavefront owns kApplyTiles tiles of 16 points
// and goes through the blocks of sixteen rows from the last up (a row needs
// only those before it), so it may overwrite them. Bound by the products (7 us
// for 64 k-points of 16 orbitals at 16^3). Vector forms waited for M's values,
// as scalar loads or from LDS, and took 25 to 44 us; row by row with separate
// input and output, and a copy back, it was 51 + 15 us.
constexpr int kApplyTiles = 4;

template <typename T>
__global__ __launch_bounds__(256) void k_apply_lower(typename Vec2<T>::type* __restrict__ w,
                                                     const double2* __restrict__ Mt, int n, int N) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, q = lane >> 4, k = blockIdx.y;
  const int p0 = (blockIdx.x * 4 + wave) * 16 * kApplyTiles;
  if (p0 >= N) return;  // uniform over the wavefront
  auto* wk = w + (size_t)k * n * N;
  const double2* Mk = Mt + (size_t)k * n * n;
  for (int r0 = (n - 1) / 16 * 16; r0 >= 0; r0 -= 16) {
    d4_t re[kApplyTiles], im[kApplyTiles];
#pragma unroll
    for (int t = 0; t < kApplyTiles; ++t) re[t] = im[t] = d4_t{0.0, 0.0, 0.0, 0.0};
    for (int j0 = 0; j0 <= r0; j0 += 16) {
      // A[row col][k q] of step s: M[r0 + col][j0 + 4 s + q], zero above the diagonal
      double mr[4], mi[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int i = r0 + col, j = j0 + 4 * s + q;
        const double2 m = Mk[(size_t)min(j, n - 1) * n + min(i, n - 1)];
        const bool in = i < n && j <= i;
        mr[s] = in ? m.x : 0.0;
        mi[s] = in ? m.y : 0.0;
      }
      typename Vec2<T>::type v[kApplyTiles][4];
#pragma unroll
      for (int t = 0; t < kApplyTiles; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          v[t][s] = wk[(size_t)min(j0 + 4 * s + q, n - 1) * N + min(p0 + 16 * t + col, N - 1)];
#pragma unroll
      for (int t = 0; t < kApplyTiles; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const bool in = j0 + 4 * s + q < n;
          const double vr = in ? (double)v[t][s].x : 0.0, vi = in ? (double)v[t][s].y : 0.0;
          re[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(mr[s], vr, re[t], 0, 0, 0);
          im[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(mr[s], vi, im[t], 0, 0, 0);
          re[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-mi[s], vi, re[t], 0, 0, 0);
          im[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(mi[s], vr, im[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < kApplyTiles; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + q + 4 * r, p = p0 + 16 * t + col;
        if (i < n && p < N) {
          typename Vec2<T>::type o;
          o.x = (T)re[t][r];
          o.y = (T)im[t][r];
          wk[(size_t)i * N + p] = o;
        }
      }
  }
}

// chunks of the grid per (k-point, tile pair): about a thousand workgroups in
// all, of at least 256 points each
static int gram_tiles(int n_orb) {
  const int t = (n_orb + 15) / 16;
  return t * (t + 1) / 2;
}
static int gram_chunk(int n_orb, int n_k, int N) {
  const long want = std::max(1L, 1024L / ((long)n_k * gram_tiles(n_orb)));
  const long pts = (N + want - 1) / want;
  return (int)std::max(256L, (pts + 63) / 64 * 64);
}
size_t gram_part_doubles(int n_orb, int n_k, int N) {
  const int chunk = gram_chunk(n_orb, n_k, N);
  return (size_t)n_k * gram_tiles(n_orb) * ((N + chunk - 1) / chunk) * 512;
}

template <typename T>
hipError_t launch_orthonormalise(typename Vec2<T>::type* w, int n_orb, int n_k, int N, double dV, double* part,
                                 double2* S, double2* Mt, int* bad, hipStream_t s) {
  const int tiles = gram_tiles(n_orb), chunk = gram_chunk(n_orb, n_k, N), nch = (N + chunk - 1) / chunk;
  hipLaunchKernelGGL((k_gram<T>), dim3((unsigned)(n_k * tiles * nch)), dim3(256), 0, s, w, n_orb, N, chunk, nch,
                     tiles, part);
  if (n_orb <= 16) {
    hipLaunchKernelGGL(k_chol_small<16>, dim3((unsigned)n_k), dim3(256), 0, s, part, n_orb, tiles, nch, dV, Mt, bad);
  } else if (n_orb <= 32) {
    hipLaunchKernelGGL(k_chol_small<32>, dim3((unsigned)n_k), dim3(256), 0, s, part, n_orb, tiles, nch, dV, Mt, bad);
  } else {
    hipLaunchKernelGGL(k_gram_reduce, dim3((unsigned)((n_orb * n_orb + 255) / 256), (unsigned)n_k), dim3(256), 0, s,
                       part, n_orb, tiles, nch, dV, S);
    hipLaunchKernelGGL(k_chol_inverse, dim3((unsigned)n_k), dim3(256), 0, s, S, Mt, n_orb, bad);
  }
  hipLaunchKernelGGL((k_apply_lower<T>), dim3((unsigned)((N + 64 * kApplyTiles - 1) / (64 * kApplyTiles)), (unsigned)n_k),
                     dim3(256), 0, s, w, Mt, n_orb, N);
  return hipGetLastError();
}
template hipError_t launch_orthonormalise<double>(double2*, int, int, int, double, double*, double2*, double2*, int*,
                                                  hipStream_t);
template hipError_t launch_orthonormalise<float>(float2*, int, int, int, double, double*, double2*, double2*, int*,
                                                 hipStream_t);

// Occupied weight kept in the reference space, per k-point:
//   S_k = sum_{m,n} |h^3 sum_r conj(ref_m(r)) w_n(r)|^2   (n_orb <= 64).
// One workgroup per k-point; the grid is walked in tiles of 16 points staged
// in LDS in FP64; thread t owns the orbital pairs t, t + 256, ... and the
// pair sums are combined by a fixed tree.
constexpr int kOvTile = 16;
constexpr int kOvMaxOrb = 64;

template <typename T>
__global__ __launch_bounds__(256) void k_overlap_weight(const typename Vec2<T>::type* __restrict__ ref,
                                                        const typename Vec2<T>::type* __restrict__ w, int n_orb,
                                                        int N, double dV, double* __restrict__ Sk) {
  __shared__ double2 tr[kOvMaxOrb][kOvTile + 1];
  __shared__ double2 tw[kOvMaxOrb][kOvTile + 1];
  __shared__ double red[256];
  constexpr int kPairs = kOvMaxOrb * kOvMaxOrb / 256;
  const int k = blockIdx.x;
  const int tid = threadIdx.x;
  const int npair = n_orb * n_orb;
  double ar[kPairs], ai[kPairs];
#pragma unroll
  for (int j = 0; j < kPairs; ++j) ar[j] = ai[j] = 0.0;
  const size_t base = (size_t)k * n_orb * N;
  for (int p0 = 0; p0 < N; p0 += kOvTile) {
    for (int t = tid; t < n_orb * kOvTile; t += 256) {
      const int m = t / kOvTile, q = t - m * kOvTile;
      const int p = p0 + q;
      double2 a = make_double2(0.0, 0.0), b = make_double2(0.0, 0.0);
      if (p < N) {
        const auto va = ref[base + (size_t)m * N + p];
        const auto vb = w[base + (size_t)m * N + p];
        a = make_double2((double)va.x, (double)va.y);
        b = make_double2((double)vb.x, (double)vb.y);
      }
      tr[m][q] = a;
      tw[m][q] = b;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
      const int pr = tid + 256 * j;
      if (pr < npair) {
        const int m = pr / n_orb, n = pr - m * n_orb;
#pragma unroll
        for (int q = 0; q < kOvTile; ++q) {
          const double2 a = tr[m][q], b = tw[n][q];
          ar[j] += a.x * b.x + a.y * b.y;  // conj(a) b
          ai[j] += a.x * b.y - a.y * b.x;
        }
      }
    }
    __syncthreads();
  }
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kPairs; ++j) s += dV * dV * (ar[j] * ar[j] + ai[j] * ai[j]);
  red[tid] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  if (tid == 0) Sk[k] = red[0];
}

template <typename T>
hipError_t launch_overlap_weight(const typename Vec2<T>::type* ref, const typename Vec2<T>::type* w, int n_orb,
                                 int n_k, int N, double dV, double* Sk, hipStream_t s) {
  if (n_orb > kOvMaxOrb) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_overlap_weight<T>), dim3((unsigned)n_k), dim3(256), 0, s, ref, w, n_orb, N, dV, Sk);
  return hipGetLastError();
}

template hipError_t launch_overlap_weight<double>(const double2*, const double2*, int, int, int, double, double*,
                                                  hipStream_t);
template hipError_t launch_overlap_weight<float>(const float2*, const float2*, int, int, int, double, double*,
                                                 hipStream_t);

}  // namespace td
