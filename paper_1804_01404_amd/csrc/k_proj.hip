// Kleinman-Bylander projections (Sec. 3.1, separable nonlocal
// pseudopotential; Sec. 4.1, phase exp(-i kappa.x) for gauge invariance):
//
//   u_{o,a,p}^{(m)} = h^3 sum_{e in sphere(a)} beta_p(x_e) (1, x, y, z)[m] exp(i kappa_k . x_e) t_o(idx_e)
//
// for every orbital o, atom a and projector p: m = 0 for the nonlocal term of
// a stage (k_project_eu), all four for the current and energy (k_project).
//
// What bounds them is the vector memory path: a sphere is some fifty runs of
// about seven points in each orbital, and every point needs its table row
// (index, two phases, four beta) besides. So a lane holds one sphere entry:
// its table row is loaded once for the kGroup orbitals of the wavefront, 64
// consecutive entries are gathered per load, and each lane keeps FP64 sums of
// its entries for every (orbital, projector) that one lane exchange per value
// adds up at the end. Laid out as a product for the FP64 matrix unit, four
// entries of eight orbitals at a time, the tables were loaded once per four
// entries and half of the lanes held copies (1.48 M vector loads for the 96
// orbitals and 256 atoms of a 96^3 cluster, each of 16 cycles: half of its
// 74 us).
//   96^3, 96 orbitals, 256 atoms, complex FP32: projection 74 -> 55 us, with the
//   previous stage's term added 136 -> 84 us (its lines alone are 230 MB), moments
//   69 -> 60 us. 36 x 40 x 27, 96 orbitals, 8 atoms, complex128: 6.3 -> 4.8, 13.1 ->
//   6.4, 8.9 -> 6.0 us.
//
// k_project writes, per orbital and atom, the nonlocal current
// sum_p 2 E_p Im(conj(v_p) u_p) (v = moments 1..3) and the nonlocal energy
// sum_p E_p |u_p|^2 into a partial table [orbital][atom][4]; k_moment_reduce
// then sums the atoms of each orbital in a fixed order.
#include "internal.h"
#include "lanes.h"

namespace td {

// The work of one wavefront: atom at, kGroup orbitals o0 .. o0 + ng - 1 of one
// k-point. SPLIT = 1: four items per workgroup, one per wavefront. SPLIT = 4
// (few items: small cells, or few orbitals over many atoms): one item per
// workgroup, its sphere entries dealt out to the four wavefronts in turn, so
// that a wavefront's serial loop over the sphere is a quarter as long. Items
// of one atom are neighbours and stay on one XCD: they share its table rows.
struct ProjItem {
  int at, k, o0, ng, sub;
  bool valid;
};
template <int SPLIT, int G>
__device__ __forceinline__ ProjItem proj_item(int n_orb, int n_orb_tot, int n_atoms) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int bid = xcd_block((int)blockIdx.x, (int)gridDim.x);
  const int item = SPLIT > 1 ? bid : bid * 4 + wave;
  const int per_k = (n_orb + G - 1) / G;
  const int n_groups = n_orb_tot / n_orb * per_k;
  ProjItem w;
  w.valid = item < n_groups * n_atoms;
  w.at = item / n_groups;
  const int grp = item - w.at * n_groups;
  w.k = grp / per_k;
  const int j0 = (grp - w.k * per_k) * G;
  w.o0 = w.k * n_orb + j0;
  w.ng = min(G, n_orb - j0);
  w.sub = SPLIT > 1 ? wave : 0;
  return w;
}

constexpr int kGroup = 4;     // orbitals of a wavefront: 32 sums
constexpr int kMomGroup = 2;  // with all four moments: 64 sums

// Stage mode: E_p u_p of every (orbital, atom, projector). ADD: the previous
// stage's nonlocal term is first added at the sphere points (in place), with
// the arithmetic of k_nl_addback (FP64 sum, one rounding to the stage
// precision); with disjoint spheres an (orbital, point) belongs to one lane.
template <typename T, int SPLIT, bool ADD>
__global__ __launch_bounds__(256) void k_project_eu(ProjArgs<T> a) {
  using T2 = typename Vec2<T>::type;
  constexpr int G = kGroup;
  __shared__ double part[SPLIT][G * 8];
  const ProjItem w = proj_item<SPLIT, G>(a.n_orb, a.n_orb_tot, a.nl.n_atoms);
  if (!w.valid) return;  // uniform over the wavefront (over the workgroup when split)
  const int lane = threadIdx.x & 63;
  const int n_atoms = a.nl.n_atoms;
  T2* __restrict__ u0 = const_cast<T2*>(a.u) + (size_t)w.o0 * a.N;
  const double2* __restrict__ phk = a.nl.phk + (size_t)w.k * a.nl.n_ent;
  const double2* __restrict__ beta = reinterpret_cast<const double2*>(a.ent_beta);
  const uniform_ptr<int> start = (uniform_ptr<int>)a.nl.atom_start;
  const int e0 = start[w.at], e1 = start[w.at + 1];
  const uniform_ptr<double> ep =
      (uniform_ptr<double>)(ADD ? reinterpret_cast<const double*>(a.Eu_prev) : nullptr);

  double acc[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[g][i] = 0.0;

  const int eb0 = e0 + 64 * w.sub;
  // the next entries' index is loaded an iteration ahead of their gathers;
  // lanes past the sphere repeat its last entry with beta = 0
  int idx = eb0 < e1 ? a.nl.ent_idx[min(eb0 + lane, e1 - 1)] : 0;
  for (int eb = eb0; eb < e1; eb += 64 * SPLIT) {
    const int e = eb + lane;
    const bool in = e < e1;
    const int ec = min(e, e1 - 1);
    T2 v[G];
#pragma unroll
    for (int g = 0; g < G; ++g) v[g] = u0[(size_t)min(g, w.ng - 1) * a.N + idx];
    const int next = a.nl.ent_idx[min(e + 64 * SPLIT, e1 - 1)];
    const double2 p1 = phk[ec], p2 = a.phA[ec];
    const double2 b01 = beta[2 * (size_t)ec], b23 = beta[2 * (size_t)ec + 1];
    const double b[kMaxProj] = {in ? b01.x : 0.0, in ? b01.y : 0.0, in ? b23.x : 0.0, in ? b23.y : 0.0};
    const double pr = p1.x * p2.x - p1.y * p2.y;
    const double pim = p1.x * p2.y + p1.y * p2.x;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (ADD) {
        const uniform_ptr<double> eg = ep + ((size_t)(w.o0 + min(g, w.ng - 1)) * n_atoms + w.at) * (2 * kMaxProj);
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int p = 0; p < kMaxProj; ++p) {
          sr += b[p] * eg[2 * p];
          si += b[p] * eg[2 * p + 1];
        }
        const double hr = pr * sr + pim * si, hi = pr * si - pim * sr;
        v[g].x += (T)(a.tau * hi + a.tau_re * hr);
        v[g].y += (T)(-a.tau * hr + a.tau_re * hi);
        if (in && g < w.ng) u0[(size_t)g * a.N + idx] = v[g];
      }
      const double ur = (double)v[g].x, ui = (double)v[g].y;
      const double wr = pr * ur - pim * ui, wi = pr * ui + pim * ur;
#pragma unroll
      for (int p = 0; p < kMaxProj; ++p) {
        acc[g][2 * p] += b[p] * wr;
        acc[g][2 * p + 1] += b[p] * wi;
      }
    }
    idx = next;
  }
  // lane l < 32 takes value l of the 32 (orbital l / 8, projector, part)
  double s[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = acc[2 * h + (i >> 3)][i & 7];
    s[h] = wave_sum16(v, lane);
  }
  int l = (lane >> 2) + 16 * (lane & 1);
  double tot = (lane & 1) ? s[1] : s[0];
  bool mine = (lane & 2) == 0;
  if (SPLIT > 1) {
    if (mine) part[w.sub][l] = tot;
    __syncthreads();
    l = threadIdx.x;
    mine = l < G * 8;
    if (!mine) return;
    tot = part[0][l];
#pragma unroll
    for (int j = 1; j < SPLIT; ++j) tot += part[j][l];
  }
  const int g = l >> 3, i = l & 7;
  if (mine && g < w.ng)
    reinterpret_cast<double*>(a.Eu)[((size_t)(w.o0 + g) * n_atoms + w.at) * (2 * kMaxProj) + i] =
        a.nl.atom_E[w.at * kMaxProj + (i >> 1)] * (a.dV * tot);
}

// Moment mode: the current and energy partials of every (orbital, atom)
template <typename T, int SPLIT>
__global__ __launch_bounds__(256) void k_project(ProjArgs<T> a) {
  using T2 = typename Vec2<T>::type;
  constexpr int G = kMomGroup;
  constexpr int V = 2 * kCols;  // sums per orbital: (projector, moment, part)
  __shared__ double part[4][G * V];
  const ProjItem w = proj_item<SPLIT, G>(a.n_orb, a.n_orb_tot, a.nl.n_atoms);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n_atoms = a.nl.n_atoms;
  if (w.valid) {
    const T2* __restrict__ u0 = a.u + (size_t)w.o0 * a.N;
    const double2* __restrict__ phk = a.nl.phk + (size_t)w.k * a.nl.n_ent;
    const double2* __restrict__ beta = reinterpret_cast<const double2*>(a.ent_beta);
    const uniform_ptr<int> start = (uniform_ptr<int>)a.nl.atom_start;
    const int e0 = start[w.at], e1 = start[w.at + 1];
    double acc[G][V];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int i = 0; i < V; ++i) acc[g][i] = 0.0;
    const int eb0 = e0 + 64 * w.sub;
    int idx = eb0 < e1 ? a.nl.ent_idx[min(eb0 + lane, e1 - 1)] : 0;
    for (int eb = eb0; eb < e1; eb += 64 * SPLIT) {
      const int e = eb + lane;
      const bool in = e < e1;
      const int ec = min(e, e1 - 1);
      T2 v[G];
#pragma unroll
      for (int g = 0; g < G; ++g) v[g] = u0[(size_t)min(g, w.ng - 1) * a.N + idx];
      const int next = a.nl.ent_idx[min(e + 64 * SPLIT, e1 - 1)];
      const double2 p1 = phk[ec], p2 = a.phA[ec];
      const double2 b01 = beta[2 * (size_t)ec], b23 = beta[2 * (size_t)ec + 1];
      const double x[3] = {a.ent_x[3 * (size_t)ec], a.ent_x[3 * (size_t)ec + 1], a.ent_x[3 * (size_t)ec + 2]};
      const double b[kMaxProj] = {in ? b01.x : 0.0, in ? b01.y : 0.0, in ? b23.x : 0.0, in ? b23.y : 0.0};
      const double pr = p1.x * p2.x - p1.y * p2.y;
      const double pim = p1.x * p2.y + p1.y * p2.x;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const double ur = (double)v[g].x, ui = (double)v[g].y;
        const double wr = pr * ur - pim * ui, wi = pr * ui + pim * ur;
#pragma unroll
        for (int m = 0; m < kMoments; ++m) {
          const double mr = m ? x[m - 1] * wr : wr, mi = m ? x[m - 1] * wi : wi;
#pragma unroll
          for (int p = 0; p < kMaxProj; ++p) {
            acc[g][2 * (p * kMoments + m)] += b[p] * mr;
            acc[g][2 * (p * kMoments + m) + 1] += b[p] * mi;
          }
        }
      }
      idx = next;
    }
    // lane l takes value l of the 64 (orbital, projector, moment, part)
    double tot = 0.0;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      double v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = acc[h >> 1][16 * (h & 1) + i];
      const double s = wave_sum16(v, lane);
      tot = (lane & 3) == h ? s : tot;
    }
    part[wave][16 * (lane & 3) + (lane >> 2)] = tot;
  }
  __syncthreads();
  // thread (item, orbital, slot): the item's sums over its SPLIT wavefronts
  constexpr int items = 4 / SPLIT;
  const int t = threadIdx.x & 63;
  if (!w.valid || t >= G * 4 || (SPLIT > 1 && wave != 0)) return;
  const int g = t >> 2, slot = t & 3;
  if (g >= w.ng) return;
  const int first = items > 1 ? wave : 0;
  auto sum = [&](int i) -> double {
    double s = part[first][g * V + i];
    for (int j = 1; j < SPLIT; ++j) s += part[j][g * V + i];
    return a.dV * s;
  };
  double r = 0.0;
#pragma unroll
  for (int p = 0; p < kMaxProj; ++p) {
    const double E = a.nl.atom_E[w.at * kMaxProj + p];
    const double ur = sum(2 * p * kMoments), ui = sum(2 * p * kMoments + 1);
    if (slot == 3) {
      r += E * (ur * ur + ui * ui);
    } else {
      const double vr = sum(2 * (p * kMoments + slot + 1)), vi = sum(2 * (p * kMoments + slot + 1) + 1);
      r += 2.0 * E * (vr * ui - vi * ur);  // 2 E_p Im(conj(v) u)
    }
  }
  reinterpret_cast<double*>(a.Eu)[((size_t)(w.o0 + g) * n_atoms + w.at) * 4 + slot] = r;
}

// jnl[o][slot] = sum over atoms of the moment-mode partials: a wavefront per
// orbital, lane 4 a + slot summing atoms a, a + 16, ... in order (one 512-byte
// row of the table per load), then the sixteen lanes of a slot in a fixed
// tree. A thread per sum walked the table alone: 33 us for 96 orbitals of 256
// atoms on two workgroups, 4 us this way.
__global__ __launch_bounds__(256) void k_moment_reduce(const double* __restrict__ part, int n_atoms, int n_orb_tot,
                                                       double* __restrict__ jnl) {
  const int lane = threadIdx.x & 63;
  const int o = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (o >= n_orb_tot) return;
  const int n = 4 * n_atoms;
  const double* __restrict__ row = part + (size_t)o * n;
  double s = 0.0;
  constexpr int kPipe = 4;
  for (int i = lane; i < n; i += 64 * kPipe) {
    double v[kPipe];
#pragma unroll
    for (int u = 0; u < kPipe; ++u) v[u] = row[min(i + 64 * u, n - 1)];
#pragma unroll
    for (int u = 0; u < kPipe; ++u) s += i + 64 * u < n ? v[u] : 0.0;
  }
#pragma unroll
  for (int off = 32; off >= 4; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane < 4) jnl[4 * o + lane] = s;
}

// Moment mode uses Eu (free between the last stage and the next step's first
// projection) as its [orbital][atom][4] partial table.
template <typename T>
hipError_t launch_project(const ProjArgs<T>& a, hipStream_t s) {
  const int G = a.moments ? kMomGroup : kGroup;
  const long total = (long)(a.n_orb_tot / a.n_orb) * ((a.n_orb + G - 1) / G) * a.nl.n_atoms;
  if (total == 0) return hipSuccess;
  // split an item over a workgroup while whole items would leave wavefront
  // slots free (1024 SIMDs of at least four)
  const bool split = total < 4096;
  const dim3 grid((unsigned)(split ? total : (total + 3) / 4)), block(256);
  if (!a.moments) {
    const bool add = a.Eu_prev != nullptr;
    if (split && add) hipLaunchKernelGGL((k_project_eu<T, 4, true>), grid, block, 0, s, a);
    else if (split) hipLaunchKernelGGL((k_project_eu<T, 4, false>), grid, block, 0, s, a);
    else if (add) hipLaunchKernelGGL((k_project_eu<T, 1, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_project_eu<T, 1, false>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  if (split) hipLaunchKernelGGL((k_project<T, 4>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_project<T, 1>), grid, block, 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_moment_reduce, dim3((unsigned)((a.n_orb_tot + 3) / 4)), dim3(256), 0, s,
                     reinterpret_cast<const double*>(a.Eu), a.nl.n_atoms, a.n_orb_tot, a.jnl);
  return hipGetLastError();
}

template hipError_t launch_project<double>(const ProjArgs<double>&, hipStream_t);
template hipError_t launch_project<float>(const ProjArgs<float>&, hipStream_t);

typedef double d4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Unit check of the lane layout of v_mfma_f64_16x16x4f64: D = A B for A [16 x 4],
// B [4 x 16] given row-major on the device; used only by a test entry point.
//   A: lane l holds A[l % 16][l / 16];  B: lane l holds B[l / 16][l % 16];
//   D: register r of lane l holds D[l / 16 + 4 r][l % 16], r = 0..3.
__global__ void k_mfma_layout(const double* A, const double* B, double* D) {
  const int l = threadIdx.x;
  const double av = A[(l % 16) * 4 + l / 16];
  const double bv = B[(l / 16) * 16 + l % 16];
  d4_t acc = {0.0, 0.0, 0.0, 0.0};
  acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
  for (int r = 0; r < 4; ++r) D[(l / 16 + 4 * r) * 16 + l % 16] = acc[r];
}

// D_b = A_b B_b for the four 4 x 4 blocks of v_mfma_f64_4x4x4f64, A, B, D
// given as [4 blocks][4][4] row-major; used only by a test entry point.
__global__ void k_mfma44_layout(const double* A, const double* B, double* D) {
  const int l = threadIdx.x;
  const int b = (l >> 2) & 3;
  const double av = A[b * 16 + (l & 3) * 4 + (l >> 4)];
  const double bv = B[b * 16 + (l >> 4) * 4 + (l & 3)];
  const double d = __builtin_amdgcn_mfma_f64_4x4x4f64(av, bv, 0.0, 0, 0, 0);
  D[b * 16 + (l >> 4) * 4 + (l & 3)] = d;
}

}  // namespace td

extern "C" int tddft_test_mfma44_layout(const double* A, const double* B, double* D) {
  double *dA, *dB, *dD;
  if (hipMalloc(&dA, 64 * sizeof(double)) != hipSuccess) return 1;
  if (hipMalloc(&dB, 64 * sizeof(double)) != hipSuccess) return 1;
  if (hipMalloc(&dD, 64 * sizeof(double)) != hipSuccess) return 1;
  hipError_t e = hipMemcpy(dA, A, 64 * sizeof(double), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(dB, B, 64 * sizeof(double), hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(td::k_mfma44_layout, dim3(1), dim3(64), 0, 0, dA, dB, dD);
    e = hipMemcpy(D, dD, 64 * sizeof(double), hipMemcpyDeviceToHost);
  }
  hipFree(dA);
  hipFree(dB);
  hipFree(dD);
  return e == hipSuccess ? 0 : 2;
}

extern "C" int tddft_test_mfma_layout(const double* A, const double* B, double* D) {
  double *dA, *dB, *dD;
  if (hipMalloc(&dA, 64 * sizeof(double)) != hipSuccess) return 1;
  if (hipMalloc(&dB, 64 * sizeof(double)) != hipSuccess) return 1;
  if (hipMalloc(&dD, 256 * sizeof(double)) != hipSuccess) return 1;
  hipMemcpy(dA, A, 64 * sizeof(double), hipMemcpyHostToDevice);
  hipMemcpy(dB, B, 64 * sizeof(double), hipMemcpyHostToDevice);
  hipLaunchKernelGGL(td::k_mfma_layout, dim3(1), dim3(64), 0, 0, dA, dB, dD);
  hipError_t e = hipMemcpy(D, dD, 256 * sizeof(double), hipMemcpyDeviceToHost);
  hipFree(dA);
  hipFree(dB);
  hipFree(dD);
  return e == hipSuccess ? 0 : 2;
}
