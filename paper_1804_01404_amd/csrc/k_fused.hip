// Whole time step of one orbital with the orbital resident in LDS.
//
// For cubic cells whose orbital fits in LDS (n = 12, 16, 20 or 24 per axis,
// N * sizeof(complex) + tables <= 160 KB), one workgroup owns one orbital and
// runs all four Horner stages u_{s-1} = w + (-i dt / s) h u_s, s = 4..1
// (Program Summary: fourth-order truncated Taylor expansion; Sec. 4.1,
// Eq. TDKS_solid for h), with
//   * u_s in LDS; u_{s-1} in registers. A thread owns a tile of four
//     consecutive x by ZR consecutive z points (see stencil_tile), so that
//     every LDS access is a 16-byte one and a value read once serves up to
//     nine outputs;
//   * the Kleinman-Bylander projections u_p = <beta_p^kappa|u_s> of every atom
//     formed in the workgroup before each stage (one wavefront per atom,
//     fixed-order reductions by register exchanges, FP64) and added back by a scatter over
//     each atom's sphere into the LDS copy (atoms coloured so that spheres of
//     one colour are disjoint: no atomics, a fixed summation order);
//   * after the last stage: w_new written once, then the observables of
//     w_new that the current needs (norm and momentum, FP64 accumulation) and
//     the moment projections for the nonlocal current at t_{n+1}.
// Traffic per orbital point and step: w is read into LDS and again as the
// Horner base of each of the four stages, w_new is written once. The orbitals
// in flight outgrow the L2s, so the later reads pass them too (20^3 x 512 k in
// complex FP32: 2.57 GB read and 0.53 GB written a launch, 2.95 times one read
// and one write; the counters do not tell the memory-side cache from HBM).
#include "internal.h"
#include "lanes.h"

namespace td {

// Global-memory views of the argument pointers. The persistent kernel reads
// its arguments from a device array, and a pointer loaded from memory is a
// generic (flat) pointer to the compiler; flat accesses also count on the LDS
// counter, so every LDS wait would wait for them. Accesses through these
// views are plain global (or scalar) loads and stores.
// (The host pass of this single-source file also parses the device templates;
// the address space exists only in the device pass.)
#if defined(__HIP_DEVICE_COMPILE__)
template <class X>
using gp = __attribute__((address_space(1))) X*;
#else
template <class X>
using gp = X*;
#endif
template <class X>
__device__ __forceinline__ gp<X> G(X* p) {
  return (gp<X>)p;
}

// E . r of the length gauge at the tile's first point and its steps along x and z
template <typename T>
struct FieldE {
  T ext, ex, ez;
};

// The k-point's row of coefficients. Each part of the stencil reads the eight
// weights of its axis with scalar loads where it needs them: all 25 held at
// once (50 scalar registers in FP64) were spilled into vector lanes and read
// back lane by lane.
#if defined(__HIP_DEVICE_COMPILE__)
template <class X>
using cp = const __attribute__((address_space(4))) X*;
#else
template <class X>
using cp = const X*;
#endif
template <typename T>
__device__ __forceinline__ cp<T> fresh(cp<T> p) {
  asm volatile("" : "+s"(p));
  return p;
}
template <typename T>
struct Axis {
  T c[4], b[4];
};
template <typename T>
__device__ __forceinline__ Axis<T> axis_coef(cp<T> row, int axis) {
  const cp<T> p = fresh<T>(row) + 8 * axis;
  Axis<T> a;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    a.c[m] = p[m];
    a.b[m] = p[kCoefB + m];
  }
  return a;
}

__device__ __forceinline__ float fmad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }

// four consecutive x points, moved as 16-byte accesses
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef double d4_t __attribute__((ext_vector_type(4)));
typedef double d2_t __attribute__((ext_vector_type(2)));
template <typename T> struct Four;
template <> struct Four<float> { using type = f4_t; };
template <> struct Four<double> { using type = d4_t; };
template <typename T>
struct Quad {
  typename Four<T>::type re, im;
};

template <typename P>
__device__ __forceinline__ Quad<float> load_quad(P p, float) {
  const f4_t a = p[0], b = p[1];
  return Quad<float>{f4_t{a.x, a.z, b.x, b.z}, f4_t{a.y, a.w, b.y, b.w}};
}
template <typename P>
__device__ __forceinline__ Quad<double> load_quad(P p, double) {
  const d2_t a = p[0], b = p[1], c = p[2], d = p[3];
  return Quad<double>{d4_t{a.x, b.x, c.x, d.x}, d4_t{a.y, b.y, c.y, d.y}};
}
template <typename P>
__device__ __forceinline__ void store_quad(P p, const Quad<float>& q) {
  p[0] = f4_t{q.re.x, q.im.x, q.re.y, q.im.y};
  p[1] = f4_t{q.re.z, q.im.z, q.re.w, q.im.w};
}
template <typename P>
__device__ __forceinline__ void store_quad(P p, const Quad<double>& q) {
  p[0] = d2_t{q.re.x, q.im.x};
  p[1] = d2_t{q.re.y, q.im.y};
  p[2] = d2_t{q.re.z, q.im.z};
  p[3] = d2_t{q.re.w, q.im.w};
}
template <typename V, typename T>
__device__ __forceinline__ V fma4(T a, V b, V c) {
  // element by element: a splat of a scalar-register weight would be copied
  return V{fmad(a, b.x, c.x), fmad(a, b.y, c.y), fmad(a, b.z, c.z), fmad(a, b.w, c.w)};
}
// 16-byte elements of the arrays: two complex FP32 or one complex FP64
template <typename T> struct Wide;
template <> struct Wide<float> { using type = f4_t; };
template <> struct Wide<double> { using type = d2_t; };

// Places (in quads of four x points) a thread's tile reads: its own first quad, the quads
// left and right of it, the rows y +- m, and the groups of ZR planes that hold
// the planes z0 - 4 .. z0 - 1 and z0 + ZR .. z0 + ZR + 3. All wrap (periodic);
// the *ok bits are clear where an isolated box has nothing (read as zero).
template <int ZR>
struct TileAt {
  static constexpr int kGroups = 4 / ZR;  // plane groups on either side
  int own, xl, xr, yp[4], ym[4], zl[kGroups], zr[kGroups];
  unsigned ok;  // bit 0 xl, 1 xr, 2..5 yp, 6..9 ym, 10.. zl, 14.. zr
};

template <int N, int ZR>
__device__ __forceinline__ TileAt<ZR> tile_at(int t) {
  constexpr int Q = N / 4, plane = N * Q;
  TileAt<ZR> a;
  const int qx = t % Q, r = t / Q, y = r % N, zb = r / N, z0 = zb * ZR;
  const int col = y * Q + qx;
  unsigned ok = 0;
  a.own = z0 * plane + col;
  a.xl = a.own + (qx > 0 ? -1 : Q - 1);
  a.xr = a.own + (qx < Q - 1 ? 1 : 1 - Q);
  ok |= (qx > 0 ? 1u : 0u) | (qx < Q - 1 ? 2u : 0u);
#pragma unroll
  for (int m = 1; m <= 4; ++m) {
    const int yp = y + m, ym = y - m;
    a.yp[m - 1] = a.own + (yp < N ? m : m - N) * Q;
    a.ym[m - 1] = a.own + (ym >= 0 ? -m : N - m) * Q;
    ok |= (yp < N ? 1u : 0u) << (1 + m) | (ym >= 0 ? 1u : 0u) << (5 + m);
  }
#pragma unroll
  for (int g = 0; g < TileAt<ZR>::kGroups; ++g) {
    const int zl = z0 - 4 + g * ZR, zr = z0 + ZR + g * ZR;
    a.zl[g] = (zl >= 0 ? zl : zl + N) * plane + col;
    a.zr[g] = (zr < N ? zr : zr - N) * plane + col;
    ok |= (zl >= 0 ? 1u : 0u) << (10 + g) | (zr < N ? 1u : 0u) << (14 + g);
  }
  a.ok = ok;
  return a;
}

// A copy of a thread's tile number that the compiler cannot see through: the
// places are rebuilt from it per stage instead of being held in registers
// across the nonlocal phases.
__device__ __forceinline__ int opaque_i(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The orbital in LDS. A quad's 16-byte words (real parts, then imaginary
// parts) lie in arrays of their own, so that a wavefront's access to one word
// of neighbouring quads is contiguous; interleaved quads (a 32- or 64-byte
// stride between lanes) conflicted on every second access: 205 M conflict
// cycles per launch of the 20^3 x 512-k cell, more than half of the LDS time.
// Every array ends with a zero word: the quad read where an isolated box ends.
template <typename T, int N>
struct LdsOrb {
  using V = typename Wide<T>::type;
  static constexpr int kQuads = N * N * N / 4;
  static constexpr int kStride = kQuads + 1;
  static constexpr int kWords = (int)(2 * sizeof(T) / 4);
  static constexpr size_t kBytes = (size_t)kWords * kStride * 16;
  V* w;

  template <bool PERIODIC>
  __device__ __forceinline__ Quad<T> quad(int place, bool in) const {
    // opaque: the compiler would otherwise load both and select every value
    if (!PERIODIC) place = opaque_i(in ? place : kQuads);
    return get(place, T(0));
  }
  __device__ __forceinline__ Quad<float> get(int q, float) const { return Quad<float>{w[q], w[kStride + q]}; }
  __device__ __forceinline__ Quad<double> get(int q, double) const {
    const d2_t a = w[q], b = w[kStride + q], c = w[2 * kStride + q], d = w[3 * kStride + q];
    return Quad<double>{d4_t{a.x, a.y, b.x, b.y}, d4_t{c.x, c.y, d.x, d.y}};
  }
  __device__ __forceinline__ void set(int q, const Quad<float>& v) const {
    w[q] = v.re;
    w[kStride + q] = v.im;
  }
  __device__ __forceinline__ void set(int q, const Quad<double>& v) const {
    w[q] = d2_t{v.re.x, v.re.y};
    w[kStride + q] = d2_t{v.re.z, v.re.w};
    w[2 * kStride + q] = d2_t{v.im.x, v.im.y};
    w[3 * kStride + q] = d2_t{v.im.z, v.im.w};
  }
  // one point: its real part; the imaginary part lies kImag further on
  static constexpr int kImag = (kWords / 2) * kStride * (int)(16 / sizeof(T));
  __device__ __forceinline__ T* point(int i) const {
    T* p = reinterpret_cast<T*>(w);
    return sizeof(T) == 4 ? p + i : p + 2 * ((i >> 2) + ((i >> 1) & 1) * kStride) + (i & 1);
  }
};

// the four points starting m (0 < m <= 4) right of a's first, out of eight
template <int M, typename V>
__device__ __forceinline__ V window(V a, V b) {
  return __builtin_shufflevector(a, b, M, M + 1, M + 2, M + 3);
}

// acc += c (p + n) + b (...): the pair of neighbours at one distance of an
// axis, weights c of the Laplacian and b of the kappa term
template <typename T>
__device__ __forceinline__ void add_pair(Quad<T>& t, T c, T b, const Quad<T>& p, const Quad<T>& n) {
  t.re = fma4(c, p.re + n.re, t.re);
  t.re = fma4(b, p.im - n.im, t.re);
  t.im = fma4(c, p.im + n.im, t.im);
  t.im = fma4(-b, p.re - n.re, t.im);
}
template <int M, typename T>
__device__ __forceinline__ void add_x_pair(Quad<T>& t, T c, T b, const Quad<T>& l, const Quad<T>& o, const Quad<T>& r) {
  add_pair<T>(t, c, b, Quad<T>{window<M>(o.re, r.re), window<M>(o.im, r.im)},
              Quad<T>{window<4 - M>(l.re, o.re), window<4 - M>(l.im, o.im)});
}

// h u_s (local part) and the Horner update of one tile of 4 x ZR points.
// Along z each plane's quad is read once and added to every output row it
// reaches; per row the y rows come in pairs and the x neighbours from three
// quads: 14, 16 and 19 quads read per row of four points for ZR = 4, 2 and 1,
// where point by point it would be 25 reads a point. The far (small) weights
// are added first and the diagonal last, so few roundings fall on the large
// partial sums (errors against 64 bits as before: 4.0e-8 of the density after
// 20 mixed steps of 20^3 x 512 k).
// Bound: vector issue in complex FP32 (632 M wave instructions per launch of
// the 20^3 x 512-k cell, 0.86 of one per CU and clock), LDS and issue together
// in complex128. A launch took 1.53 ms (FP32; 817 M instructions) and 0.44 ms
// (complex128, 64 k) when a thread owned a whole column of points read one by
// one with the last wavefronts idle; now 1.21 and 0.32 ms; 16^3 x 64 k 0.136 ->
// 0.122 and 0.290 -> 0.183 ms, 24^3 x 27 k (FP32) 0.229 -> 0.144 ms.
template <typename T, int N, int ZR, bool PERIODIC, bool IMAG>
__device__ __forceinline__ void stencil_tile(const LdsOrb<T, N> u, gp<const T> V, cp<T> row, const FieldE<T>& fe,
                                             const TileAt<ZR>& at, gp<const typename Vec2<T>::type> wg,
                                             Quad<T> (&un)[ZR], T tau) {
  constexpr int plane = N * N / 4;  // quads
  using V16 = typename Wide<T>::type;
  using V4 = typename Four<T>::type;
  const V4 zero = (V4)(T(0));
#pragma unroll
  for (int r = 0; r < ZR; ++r) un[r].re = un[r].im = zero;
  const Axis<T> az = axis_coef<T>(row, 2);
  // planes z0 - 4 .. z0 + ZR + 3 in order
#pragma unroll
  for (int p = -4; p < ZR + 4; ++p) {
    if (ZR == 1 && p == 0) continue;
    int place;
    bool in = true;
    if (p < 0) {
      const int g = (p + 4) / ZR;
      place = at.zl[g] + ((p + 4) % ZR) * plane;
      in = at.ok >> (10 + g) & 1;
    } else if (p < ZR) {
      place = at.own + p * plane;
    } else {
      const int g = (p - ZR) / ZR;
      place = at.zr[g] + ((p - ZR) % ZR) * plane;
      in = at.ok >> (14 + g) & 1;
    }
    const Quad<T> q = u.template quad<PERIODIC>(place, in);
#pragma unroll
    for (int r = 0; r < ZR; ++r) {
      const int d = p - r;
      if (d == 0 || d > 4 || d < -4) continue;
      const int m = (d > 0 ? d : -d) - 1;
      const T b = d > 0 ? az.b[m] : -az.b[m];
      un[r].re = fma4(b, q.im, fma4(az.c[m], q.re, un[r].re));
      un[r].im = fma4(-b, q.re, fma4(az.c[m], q.im, un[r].im));
    }
    if ((p & 1) || sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
  }
  Axis<T> ax, ay;
  if (sizeof(T) == 4) {
    ay = axis_coef<T>(row, 1);
    ax = axis_coef<T>(row, 0);
  }
#pragma unroll
  for (int r = 0; r < ZR; ++r) {
    const int off = at.own + r * plane;
    V4 v;
    Quad<T> w;
    // w is re-read (from cache) rather than held in registers for all stages;
    // in FP64 it is loaded after the neighbours, for the registers' sake
    auto load_w = [&]() __attribute__((always_inline)) {
      v = *(gp<const V4>)(V + 4 * off);
      w = load_quad((gp<const V16>)(wg + 4 * off), T(0));
    };
    if (sizeof(T) == 4) load_w();
    Quad<T> t{zero, zero};
    if (sizeof(T) == 8) ay = axis_coef<T>(row, 1);
#pragma unroll
    for (int m = 3; m >= 0; --m) {
      const Quad<T> p = u.template quad<PERIODIC>(at.yp[m] + r * plane, at.ok >> (2 + m) & 1);
      const Quad<T> n = u.template quad<PERIODIC>(at.ym[m] + r * plane, at.ok >> (6 + m) & 1);
      add_pair<T>(t, ay.c[m], ay.b[m], p, n);
      if (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
    }
    const Quad<T> c = u.template quad<true>(off, true);
    const Quad<T> xl = u.template quad<PERIODIC>(at.xl + r * plane, at.ok & 1);
    const Quad<T> xr = u.template quad<PERIODIC>(at.xr + r * plane, at.ok >> 1 & 1);
    if (sizeof(T) == 8) ax = axis_coef<T>(row, 0);
    add_x_pair<4>(t, ax.c[3], ax.b[3], xl, c, xr);
    add_x_pair<3>(t, ax.c[2], ax.b[2], xl, c, xr);
    add_x_pair<2>(t, ax.c[1], ax.b[1], xl, c, xr);
    add_x_pair<1>(t, ax.c[0], ax.b[0], xl, c, xr);
    if (sizeof(T) == 8) {
      __builtin_amdgcn_sched_barrier(0);
      load_w();
    }
    V4 dg = v + row[kCoefDiag];
    if (!PERIODIC) dg += (V4)(fe.ext + fe.ez * (T)r) + V4{T(0), fe.ex, 2 * fe.ex, 3 * fe.ex};
    const V4 hr = __builtin_elementwise_fma(dg, c.re, un[r].re + t.re);
    const V4 hi = __builtin_elementwise_fma(dg, c.im, un[r].im + t.im);
    if (IMAG) {  // u_{s-1} = w - tau h u_s
      un[r].re = fma4(-tau, hr, w.re);
      un[r].im = fma4(-tau, hi, w.im);
    } else {
      un[r].re = fma4(tau, hi, w.re);
      un[r].im = fma4(-tau, hr, w.im);
    }
    // one row at a time: bounds the loads in flight and so the registers
    __builtin_amdgcn_sched_barrier(0);
  }
}

// norm and momentum sums of w_new over one tile: the weighted neighbour sums
// in the stage precision, their products with w and the running sums in FP64
// (as in the streaming observables kernel)
template <typename T, int N, int ZR, bool PERIODIC>
__device__ __forceinline__ void observe_tile(const LdsOrb<T, N> u, const T (&dw)[3][4],
                                             const TileAt<ZR>& at, double (&sv)[4]) {
  // Summed over the whole grid, Im(conj(w) D w) with the antisymmetric
  // difference D = sum_m d_m (S_m - S_-m) equals 2 sum_m d_m Im(conj(w) S_m w)
  // (shift r -> r - m in the backward half; zero outside an isolated box), so
  // each point needs only its forward neighbours.
  constexpr int plane = N * N / 4;  // quads
  using V4 = typename Four<T>::type;
  const V4 zero = (V4)(T(0));
#pragma unroll
  for (int r = 0; r < ZR; ++r) {
    const int off = at.own + r * plane;
    const Quad<T> c = u.template quad<true>(off, true);
    Quad<T> s{zero, zero};
    auto add = [&](T d, V4 re, V4 im) __attribute__((always_inline)) {
      s.re = fma4(d, re, s.re);
      s.im = fma4(d, im, s.im);
    };
    auto take = [&](int axis) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        sv[1 + axis] = fmad((double)c.re[i], (double)s.im[i], fmad(-(double)c.im[i], (double)s.re[i], sv[1 + axis]));
      s.re = s.im = zero;
    };
    const Quad<T> xr = u.template quad<PERIODIC>(at.xr + r * plane, at.ok >> 1 & 1);
    add(dw[0][3], xr.re, xr.im);
    add(dw[0][2], window<3>(c.re, xr.re), window<3>(c.im, xr.im));
    add(dw[0][1], window<2>(c.re, xr.re), window<2>(c.im, xr.im));
    add(dw[0][0], window<1>(c.re, xr.re), window<1>(c.im, xr.im));
    take(0);
#pragma unroll
    for (int m = 3; m >= 0; --m) {
      const Quad<T> q = u.template quad<PERIODIC>(at.yp[m] + r * plane, at.ok >> (2 + m) & 1);
      add(dw[1][m], q.re, q.im);
      if (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
    }
    take(1);
#pragma unroll
    for (int m = 3; m >= 0; --m) {
      const int p = r + m + 1;
      if (p < ZR) {
        const Quad<T> q = u.template quad<true>(at.own + p * plane, true);
        add(dw[2][m], q.re, q.im);
      } else {
        const int g = (p - ZR) / ZR;
        const Quad<T> q = u.template quad<PERIODIC>(at.zr[g] + ((p - ZR) % ZR) * plane, at.ok >> (14 + g) & 1);
        add(dw[2][m], q.re, q.im);
      }
      if (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
    }
    take(2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double cr = (double)c.re[i], ci = (double)c.im[i];
      sv[0] = fmad(cr, cr, fmad(ci, ci, sv[0]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ITEMS: the body runs once per item of a loop (the persistent form); IMAG:
// imaginary time (dt is the real step of exp(-dt h)), no observables
template <typename T, int N, int ZR, bool PERIODIC, bool ITEMS = false, bool IMAG = false>
__device__ __forceinline__ void fused_body(const FusedArgs<T>& a, const int o, unsigned char* smem_raw) {
  using T2 = typename Vec2<T>::type;
  using V16 = typename Wide<T>::type;
  constexpr int plane = N * N / 4;  // quads
  constexpr int NP = N * N * N;
  constexpr int TILES = NP / (4 * ZR);
  const int n_atoms = a.nl.n_atoms;
  const int S = a.nl.n_ent;
  const gp<const int> atom_start = G(a.nl.atom_start);
  const gp<const int> ent_idx = G(a.nl.ent_idx);
  const gp<const double> atom_E = G(a.nl.atom_E);
  const gp<const double> ent_beta = G(a.ent_beta);
  const gp<const double> ent_x = G(a.ent_x);
  const gp<const int> color_start = G(a.color_start);
  const gp<const int> color_atoms = G(a.color_atoms);
  const gp<const double2> phAJ = G(a.phAJ);
  const LdsOrb<T, N> u{reinterpret_cast<V16*>(smem_raw)};
  double2* eu = reinterpret_cast<double2*>(smem_raw + LdsOrb<T, N>::kBytes);  // [n_atoms][4]
  double* red = reinterpret_cast<double*>(eu + (size_t)n_atoms * kMaxProj);   // [16][4]
  double* ja = red + 16 * 4;                                                  // [n_atoms][4]

  const int k = o / a.g.n_orb;
  // in the persistent form the thread index is opaque to the compiler, so
  // that the values derived from it are formed per item instead of being
  // hoisted out of the item loop and held in registers across it
  int tid = threadIdx.x;
  if (ITEMS) asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = tid >> 6, nwaves = blockDim.x >> 6;
  const bool active = tid < TILES;
  const int tile = active ? tid : 0;

  if (!PERIODIC && tid == 0) u.set(LdsOrb<T, N>::kQuads, Quad<T>{});
  const gp<T2> wg = G(a.w) + (size_t)o * NP;
  if (active) {
    const int own = tile_at<N, ZR>(tile).own;
#pragma unroll
    for (int r = 0; r < ZR; ++r)
      u.set(own + r * plane, load_quad((gp<const V16>)(wg + 4 * (own + r * plane)), T(0)));
  }

  const cp<T> row = (cp<T>)(a.coef) + (size_t)k * kCoef;
  FieldE<T> fe{0, 0, 0};
  if (!PERIODIC && a.efield) {
    // E . r with r from the box centre; the steps inside the tile are added per point
    const gp<const double> ef = G(a.efield);
    const int qx = tile % (N / 4), y = tile / (N / 4) % N, z0 = tile / (N / 4 * N) * ZR;
    fe.ext = (T)(ef[0] * (4 * qx - 0.5 * (N - 1)) * a.g.h1 + ef[1] * (y - 0.5 * (N - 1)) * a.g.h2 +
                 ef[2] * (z0 - 0.5 * (N - 1)) * a.g.h3);
    fe.ex = (T)(ef[0] * a.g.h1);
    fe.ez = (T)(ef[2] * a.g.h3);
  }
  const gp<const double2> phk = G(a.nl.phk) + (size_t)k * S;
  const gp<const double2> phkA = G(a.phkA) + (size_t)k * S;  // exp(i kappa . x_e) of this step
  __syncthreads();

  // ---- projections of u_s: one wavefront per atom, FP64
  auto project = [&]() {
    for (int at = wave; at < n_atoms; at += nwaves) {
      const int e0 = atom_start[at], e1 = atom_start[at + 1];
      double acc[2 * kMaxProj] = {0, 0, 0, 0, 0, 0, 0, 0};
      for (int e = e0 + lane; e < e1; e += 64) {
        const T* const pt = u.point(ent_idx[e]);
        const T vx = pt[0], vy = pt[LdsOrb<T, N>::kImag];
        const double2 ph = phkA[e];
        const double pr = ph.x, pim = ph.y;
        const double gr = pr * (double)vx - pim * (double)vy;
        const double gi = pr * (double)vy + pim * (double)vx;
#pragma unroll
        for (int p = 0; p < kMaxProj; ++p) {
          const double b = ent_beta[(size_t)e * kMaxProj + p];
          acc[2 * p] += b * gr;
          acc[2 * p + 1] += b * gi;
        }
      }
      // value 2p (real) sits in lanes 16p.., value 2p + 1 (imaginary) 8 lanes up
      const double tot = wave_sum8(acc, lane);
      const double im = dpp<kXor8>(tot);
      if ((lane & 15) == 0) {
        const int p = lane >> 4;
        const double E = atom_E[at * kMaxProj + p] * a.dV;
        eu[at * kMaxProj + p] = make_double2(E * tot, E * im);
      }
    }
    __syncthreads();
  };
  // With disjoint spheres (one colour) every sphere point belongs to one
  // atom, so the wavefront that adds an atom's nonlocal term of stage s to
  // its points can go on to form that atom's projections of the completed
  // u_{s-1} without waiting for the other atoms: one barrier fewer per stage.
  const bool one_colour = a.n_colors == 1;
  if (n_atoms > 0) project();

#pragma unroll 1
  for (int s = 4; s >= 1; --s) {
    // ---- local part of h u_s and the Horner update
    const T tau = (T)(a.dt / s);
    Quad<T> un[ZR];
    const int own = tile_at<N, ZR>(tile).own;
    if (active) stencil_tile<T, N, ZR, PERIODIC, IMAG>(u, G(a.V), row, fe, tile_at<N, ZR>(opaque_i(tile)), wg, un, tau);
    __syncthreads();
    if (active) {
#pragma unroll
      for (int r = 0; r < ZR; ++r) u.set(own + r * plane, un[r]);
    }
    __syncthreads();
    // ---- nonlocal part of the stage, scattered over each atom's sphere:
    // u_{s-1}(x_e) += (-i tau) exp(-i kappa.x_e) sum_p beta_p(x_e) E_p u_p.
    // Atoms of one colour have disjoint spheres, colours run in a fixed order.
    if (n_atoms > 0) {
      const double taud = a.dt / s;
      if (one_colour) {
        for (int at = wave; at < n_atoms; at += nwaves) {
          const int e0 = atom_start[at], e1 = atom_start[at + 1];
          double2 E4[kMaxProj];
#pragma unroll
          for (int p = 0; p < kMaxProj; ++p) E4[p] = eu[at * kMaxProj + p];
          // the completed value of a point goes straight into the next
          // stage's projection (not needed after the last one): one read of
          // the tables serves both
          double acc[2 * kMaxProj] = {0, 0, 0, 0, 0, 0, 0, 0};
          for (int e = e0 + lane; e < e1; e += 64) {
            const int idx = ent_idx[e];
            const double2 ph = phkA[e];
            const double pr = ph.x, pim = ph.y;
            double b[kMaxProj];
#pragma unroll
            for (int p = 0; p < kMaxProj; ++p) b[p] = ent_beta[(size_t)e * kMaxProj + p];
            double sr = 0.0, si = 0.0;
#pragma unroll
            for (int p = 0; p < kMaxProj; ++p) {
              sr += b[p] * E4[p].x;
              si += b[p] * E4[p].y;
            }
            const double cr = pr * sr + pim * si, ci = pr * si - pim * sr;
            T* const pt = u.point(idx);
            const T vx = pt[0] + (T)(taud * (IMAG ? -cr : ci)), vy = pt[LdsOrb<T, N>::kImag] - (T)(taud * (IMAG ? ci : cr));
            pt[0] = vx;
            pt[LdsOrb<T, N>::kImag] = vy;
            const double gr = pr * (double)vx - pim * (double)vy;
            const double gi = pr * (double)vy + pim * (double)vx;
#pragma unroll
            for (int p = 0; p < kMaxProj; ++p) {
              acc[2 * p] += b[p] * gr;
              acc[2 * p + 1] += b[p] * gi;
            }
          }
          if (s > 1) {
            const double tot = wave_sum8(acc, lane);
            const double im = dpp<kXor8>(tot);
            if ((lane & 15) == 0) {
              const int p = lane >> 4;
              const double E = atom_E[at * kMaxProj + p] * a.dV;
              eu[at * kMaxProj + p] = make_double2(E * tot, E * im);
            }
          }
        }
        __syncthreads();
      } else {
        for (int cl = 0; cl < a.n_colors; ++cl) {
          for (int ii = color_start[cl] + wave; ii < color_start[cl + 1]; ii += nwaves) {
            const int at = color_atoms[ii];
            const int e0 = atom_start[at], e1 = atom_start[at + 1];
            double2 E4[kMaxProj];
#pragma unroll
            for (int p = 0; p < kMaxProj; ++p) E4[p] = eu[at * kMaxProj + p];
            for (int e = e0 + lane; e < e1; e += 64) {
              const int idx = ent_idx[e];
              const double2 ph = phkA[e];
              const double pr = ph.x, pim = ph.y;
              double sr = 0.0, si = 0.0;
#pragma unroll
              for (int p = 0; p < kMaxProj; ++p) {
                const double b = ent_beta[(size_t)e * kMaxProj + p];
                sr += b * E4[p].x;
                si += b * E4[p].y;
              }
              const double cr = pr * sr + pim * si, ci = pr * si - pim * sr;
              T* const pt = u.point(idx);
              const T vx = pt[0] + (T)(taud * (IMAG ? -cr : ci)), vy = pt[LdsOrb<T, N>::kImag] - (T)(taud * (IMAG ? ci : cr));
              pt[0] = vx;
              pt[LdsOrb<T, N>::kImag] = vy;
            }
          }
          __syncthreads();
        }
        if (s > 1) project();
      }
    }
  }

  // ---- w_new to HBM, observables for the current
  double sv[4] = {0, 0, 0, 0};
  {
    if (active) {
      const TileAt<ZR> at = tile_at<N, ZR>(opaque_i(tile));
#pragma unroll
      for (int r = 0; r < ZR; ++r)
        store_quad((gp<V16>)(wg + 4 * (at.own + r * plane)), u.get(at.own + r * plane, T(0)));
      if (!IMAG) observe_tile<T, N, ZR, PERIODIC>(u, a.dhc, at, sv);
    }
  }
  if (IMAG) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) sv[i] = wave_sum(i == 0 ? sv[0] : 2.0 * sv[i]);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave * 4 + i] = sv[i];
  }
  __syncthreads();
  if (tid < 6) {
    double acc = 0;
    if (tid < 4)
      for (int wv = 0; wv < nwaves; ++wv) acc += red[wv * 4 + tid];
    G(a.obs)[(size_t)o * 8 + tid] = acc;  // slots 4, 5 (kinetic, local) stay 0 here
  }
  __syncthreads();

  // ---- nonlocal current and energy at t_{n+1}: moments (1, x, y, z) of the
  // projections with the phase of A_{n+1}; one wavefront per atom, two
  // moments per gather of the sphere values
  if (n_atoms > 0) {
    for (int at = wave; at < n_atoms; at += nwaves) {
      const int e0 = atom_start[at], e1 = atom_start[at + 1];
      // lane 32 mm + 8 p holds the real part of the pass's moment mm of
      // projector p and receives the imaginary part from 4 lanes up
      const int pl = (lane >> 3) & 3, mml = lane >> 5;
      const double E = atom_E[at * kMaxProj + pl];
      double ur = 0.0, ui = 0.0;
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
        // value 8 mm + 2 p + (0 real, 1 imaginary) for moments m = 2 pass + mm
        double acc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.0;
        for (int e = e0 + lane; e < e1; e += 64) {
          const T* const pt = u.point(ent_idx[e]);
          const T vx = pt[0], vy = pt[LdsOrb<T, N>::kImag];
          const double2 p1 = phk[e], p2 = phAJ[e];
          const double pr = p1.x * p2.x - p1.y * p2.y, pim = p1.x * p2.y + p1.y * p2.x;
          const double gr = pr * (double)vx - pim * (double)vy;
          const double gi = pr * (double)vy + pim * (double)vx;
          const double m0 = pass == 0 ? 1.0 : ent_x[3 * (size_t)e + 1];
          const double m1 = ent_x[3 * (size_t)e + 2 * pass];
#pragma unroll
          for (int p = 0; p < kMaxProj; ++p) {
            const double b = ent_beta[(size_t)e * kMaxProj + p];
            const double br = b * gr, bi = b * gi;
            acc[2 * p] += m0 * br;
            acc[2 * p + 1] += m0 * bi;
            acc[8 + 2 * p] += m1 * br;
            acc[8 + 2 * p + 1] += m1 * bi;
          }
        }
        const double tot = wave_sum16(acc, lane) * a.dV;
        // every quad holds its full sum, so lane ^ 7 is the other part's quad
        const double im = dpp<kXor7>(tot);
        if (pass == 0) {  // u_p of the lower half's moment 0, for both halves
          ur = swap32(tot, tot).x;
          ui = swap32(im, im).x;
        }
        // E_p |u_p|^2 for m = 0, 2 E_p Im(conj(v_p) u_p) for m = 1..3, summed over p
        const int m = 2 * pass + mml;
        double c = (m == 0) ? E * (ur * ur + ui * ui) : 2.0 * E * (tot * ui - im * ur);
        c += dpp<kXor8>(c);
        c = sum16(c);
        if ((lane & 31) == 0) ja[at * 4 + (m == 0 ? 3 : m - 1)] = c;
      }
    }
  }
  __syncthreads();
  if (tid < 4) {  // atoms summed in index order, whatever wavefront formed them
    double acc = 0;
    for (int at = 0; at < n_atoms; ++at) acc += ja[at * 4 + tid];
    G(a.jnl)[(size_t)o * 4 + tid] = acc;
  }
}

// Points along z of a thread's tile, fixed per grid size and precision so that
// every path computes the same bits; workgroup size: the tiles' threads,
// rounded up to whole wavefronts and to eight of them, so that the nonlocal
// phases (one wavefront per atom) run the eight atoms of a diamond cell side by
// side; waves per SIMD the registers have to leave room for. At 20^3 four rows
// give 500 tiles (512 threads, 64 KB, two workgroups per CU) in complex FP32
// and two rows 1000 tiles (1024 threads, 128 KB, one per CU) in complex128;
// 16^3 takes 512 and 12^3 432 tiles, 24^3 (complex FP32 only, 110 KB) 864.
__host__ __device__ constexpr int fused_rows_of(int n, size_t real) {
  return n == 12 ? 1 : (n == 16 ? 2 : (n == 20 && real == 8 ? 2 : 4));
}
template <typename T, int N>
struct FusedShape {
  static constexpr int kRows = fused_rows_of(N, sizeof(T));
  static constexpr int kTiles = N * N * N / (4 * kRows);
  static constexpr int kThreads = kTiles <= 512 ? 512 : (kTiles + 63) / 64 * 64;
  static constexpr int kWaves = 4;
};
int fused_rows(int n, size_t elem) { return fused_rows_of(n, elem / 2); }

// one orbital per workgroup
template <typename T, int N, bool PERIODIC>
__global__ __launch_bounds__((FusedShape<T, N>::kThreads), (FusedShape<T, N>::kWaves)) void k_fused(FusedArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  fused_body<T, N, FusedShape<T, N>::kRows, PERIODIC>(a, blockIdx.x, smem_raw);
}

// the imaginary-time step of the ground-state preparation: as the per-stage
// kernels (four stages of 23 us, projections of 17, the add-back) it was
// 0.19 ms for 16^3 x 64 k in complex FP32, this is 0.10 ms
template <typename T, int N, bool PERIODIC>
__global__ __launch_bounds__((FusedShape<T, N>::kThreads), (FusedShape<T, N>::kWaves)) void k_fused_imaginary(
    FusedArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  fused_body<T, N, FusedShape<T, N>::kRows, PERIODIC, false, true>(a, blockIdx.x, smem_raw);
}

// Persistent form for batches of cells with the same grid: a fixed grid of
// workgroups pulls (cell, orbital) items from a device queue in the given
// (largest-cell-first) order until the list is exhausted; every item is
// computed exactly as in k_fused, so the result does not depend on which
// workgroup takes it.
template <typename T, int N, bool PERIODIC>
__global__ __launch_bounds__((FusedShape<T, N>::kThreads), (FusedShape<T, N>::kWaves)) void k_fused_persistent(
    const FusedArgs<T>* __restrict__ cells, const int2* __restrict__ items, int n_items, int* queue) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ int next;
  if (threadIdx.x == 0) next = atomicAdd(queue, 1);
  __syncthreads();
  int it = __builtin_amdgcn_readfirstlane(next);
  __syncthreads();
  while (it < n_items) {
    // claim the following item now, so that the queue's round trip overlaps
    // this item's work (every item is still taken exactly once)
    int claim = 0;
    if (threadIdx.x == 0) claim = atomicAdd(queue, 1);
    // the cell and orbital are uniform: scalar registers, so that the
    // cell's arguments are read with scalar loads as kernel arguments are
    const int2 ci = items[it];
    const int cx = __builtin_amdgcn_readfirstlane(ci.x), orb = __builtin_amdgcn_readfirstlane(ci.y);
    fused_body<T, N, FusedShape<T, N>::kRows, PERIODIC, true>(cells[cx], orb, smem_raw);
    __syncthreads();
    if (threadIdx.x == 0) next = claim;
    __syncthreads();
    it = __builtin_amdgcn_readfirstlane(next);
    __syncthreads();
  }
}

size_t fused_lds_bytes(const Geometry& g, int n_atoms, size_t elem) {
  const size_t N = (size_t)g.n1 * g.n2 * g.n3;
  // the orbital with a zero word per 16-byte word array (LdsOrb), eu, red, ja
  return (N * elem + elem / 4 * 16) + (size_t)n_atoms * kMaxProj * sizeof(double2) + 16 * 4 * sizeof(double) +
         (size_t)n_atoms * 4 * sizeof(double);
}

bool fused_supported(const Geometry& g, int n_atoms, size_t elem) {
  const int n = g.n3;
  if (n != 12 && n != 16 && n != 20 && n != 24) return false;
  if (g.n1 != n || g.n2 != n) return false;
  return fused_lds_bytes(g, n_atoms, elem) <= 160 * 1024;
}

template <typename T, int N>
static void launch_n(bool periodic, bool imaginary, const FusedArgs<T>& a, size_t lds, hipStream_t s) {
  constexpr int threads = FusedShape<T, N>::kThreads;
  const dim3 grid((unsigned)((size_t)a.g.n_orb * a.g.n_k));
  if (periodic && !imaginary)
    hipLaunchKernelGGL((k_fused<T, N, true>), grid, dim3(threads), lds, s, a);
  else if (!imaginary)
    hipLaunchKernelGGL((k_fused<T, N, false>), grid, dim3(threads), lds, s, a);
  else if (periodic)
    hipLaunchKernelGGL((k_fused_imaginary<T, N, true>), grid, dim3(threads), lds, s, a);
  else
    hipLaunchKernelGGL((k_fused_imaginary<T, N, false>), grid, dim3(threads), lds, s, a);
}

template <typename T>
hipError_t launch_fused(const FusedArgs<T>& a, hipStream_t s, bool imaginary) {
  using T2 = typename Vec2<T>::type;
  if (!fused_supported(a.g, a.nl.n_atoms, sizeof(T2))) return hipErrorInvalidValue;
  const size_t lds = fused_lds_bytes(a.g, a.nl.n_atoms, sizeof(T2));
  const bool per = a.g.periodic != 0;
  switch (a.g.n3) {
    case 12: launch_n<T, 12>(per, imaginary, a, lds, s); break;
    case 16: launch_n<T, 16>(per, imaginary, a, lds, s); break;
    case 20: launch_n<T, 20>(per, imaginary, a, lds, s); break;
    default:
      if constexpr (sizeof(T) == 4) launch_n<T, 24>(per, imaginary, a, lds, s);  // complex128 does not fit
      break;
  }
  return hipGetLastError();
}

template hipError_t launch_fused<double>(const FusedArgs<double>&, hipStream_t, bool);
template hipError_t launch_fused<float>(const FusedArgs<float>&, hipStream_t, bool);

template <typename T, int N>
static void launch_pers_n(bool periodic, const FusedArgs<T>* cells, const int2* items, int n_items,
                          int* queue, int wgs, size_t lds, hipStream_t s) {
  constexpr int threads = FusedShape<T, N>::kThreads;
  if (periodic)
    hipLaunchKernelGGL((k_fused_persistent<T, N, true>), dim3(wgs), dim3(threads), lds, s, cells, items, n_items,
                       queue);
  else
    hipLaunchKernelGGL((k_fused_persistent<T, N, false>), dim3(wgs), dim3(threads), lds, s, cells, items, n_items,
                       queue);
}

template <typename T>
hipError_t launch_fused_persistent(int n, bool periodic, const FusedArgs<T>* cells, const int2* items, int n_items,
                                   int* queue, int wgs, size_t lds, hipStream_t s) {
  if (wgs < 1 || n_items < 1) return hipErrorInvalidValue;
  switch (n) {
    case 12: launch_pers_n<T, 12>(periodic, cells, items, n_items, queue, wgs, lds, s); break;
    case 16: launch_pers_n<T, 16>(periodic, cells, items, n_items, queue, wgs, lds, s); break;
    case 20: launch_pers_n<T, 20>(periodic, cells, items, n_items, queue, wgs, lds, s); break;
    case 24:
      if constexpr (sizeof(T) == 4) {
        launch_pers_n<T, 24>(periodic, cells, items, n_items, queue, wgs, lds, s);
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template hipError_t launch_fused_persistent<double>(int, bool, const FusedArgs<double>*, const int2*, int, int*, int,
                                                    size_t, hipStream_t);
template hipError_t launch_fused_persistent<float>(int, bool, const FusedArgs<float>*, const int2*, int, int*, int,
                                                   size_t, hipStream_t);

}  // namespace td
