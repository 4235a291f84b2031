// Kernels of the current surrogate that stands in for a microscopic cell in
// the multiscale coupling (Sec. 5): a causal window of the vector potential
// -> dense W->H, tanh -> dense H->H, tanh -> dense H->1, plus a linear skip
// W->1. FP32 throughout, the dense layers on the matrix cores; every reduction
// runs in a fixed order, so results do not depend on scheduling. Parameter layout (flat): W1 [H][W], b1 [H],
// W2 [H][H], b2 [H], w3 [H], b3 [1], ws [W]. Adam follows Kingma and Ba
// (ICLR 2015, Algorithm 1).
#include "internal.h"

namespace td {

constexpr int kTile = 16;      // output tile of one workgroup (the MFMA's 16 x 16)
constexpr int kGemmWaves = 4;  // wavefronts per tile, each a quarter of the k range

typedef float f32x4 __attribute__((ext_vector_type(4)));

// C[i][j] = sum_k A(i, k) B(k, j) for i < M, j < N, with A(i, k) = A[i*sai + k*sak]
// and B(k, j) = B[k*sbk + j*sbj]; epilogue: + bias[j] (if bias), tanh (if act),
// then * (1 - aux[i][j]^2) (if aux, the tanh derivative of a stored activation).
// On the matrix cores: v_mfma_f32_16x16x4f32 takes A(i, k) from lane i + 16 k
// and B(k, j) from lane j + 16 k of a 16 x 4 / 4 x 16 slice and leaves
// C(4 g + r, j) in element r of lane j + 16 g. Each of the four wavefronts of a
// tile runs a contiguous quarter of the k steps; the partial tiles are added in
// wavefront order, so the result does not depend on scheduling.
__global__ __launch_bounds__(kGemmWaves * 64) void k_gemm(const float* __restrict__ A, long sai, long sak,
                                                         const float* __restrict__ B, long sbk, long sbj,
                                                         float* __restrict__ C, int M, int N, int K,
                                                         const float* __restrict__ bias, int act,
                                                         const float* __restrict__ aux) {
  __shared__ float part[kGemmWaves - 1][kTile][kTile + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int i0 = blockIdx.y * kTile, j0 = blockIdx.x * kTile;
  // rows and columns past the matrix load a clamped in-range element and use 0
  const bool aok = i0 + r < M, bok = j0 + r < N;
  const long ia = min(i0 + r, M - 1), jb = min(j0 + r, N - 1);
  const int steps = (K + 3) / 4;
  const int per = (steps + kGemmWaves - 1) / kGemmWaves;
  const int s0 = wave * per, s1 = min(steps, s0 + per);
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  // chunks of kChunk k steps: every load of a chunk is issued before its
  // products (steps past s1 or K load a clamped element and use 0)
  constexpr int kChunk = 8;
  for (int c0 = s0; c0 < s1; c0 += kChunk) {
    float av[kChunk], bv[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const long kc = min(4 * (c0 + u) + q, K - 1);
      av[u] = A[ia * sai + kc * sak];
      bv[u] = B[kc * sbk + jb * sbj];
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const bool kin = c0 + u < s1 && 4 * (c0 + u) + q < K;
      const float a = (aok && kin) ? av[u] : 0.0f;
      const float b = (bok && kin) ? bv[u] : 0.0f;
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) part[wave - 1][4 * q + e][r] = acc[e];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = acc[e];
#pragma unroll
      for (int w = 0; w < kGemmWaves - 1; ++w) v += part[w][4 * q + e][r];
      const int i = i0 + 4 * q + e, j = j0 + r;
      if (i < M && j < N) {
        if (bias) v += bias[j];
        if (act) v = tanhf(v);
        if (aux) {
          const float h = aux[(long)i * N + j];
          v *= 1.0f - h * h;
        }
        C[(long)i * N + j] = v;
      }
    }
  }
}

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// y[b] = w3 . h2[b] + b3 + ws . x[b]; one wavefront per sample
__global__ void k_nn_out(const float* __restrict__ h2, const float* __restrict__ x, const float* __restrict__ w3,
                         const float* __restrict__ b3, const float* __restrict__ ws, int B, int H, int W,
                         float* __restrict__ y) {
  const int b = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (b >= B) return;
  float s = 0.0f;
  for (int h = lane; h < H; h += 64) s = fmaf(h2[(long)b * H + h], w3[h], s);
  float t = 0.0f;
  for (int w = lane; w < W; w += 64) t = fmaf(x[(long)b * W + w], ws[w], t);
  s = wave_sum_f(s) + b3[0] + wave_sum_f(t);
  if (lane == 0) y[b] = s;
}

// dy[b] = 2 (y[b] - t[b]) / B and the loss (1/B) sum (y - t)^2 (one block)
__global__ __launch_bounds__(256) void k_nn_dy_loss(const float* __restrict__ y, const float* __restrict__ t, int B,
                                                    float* __restrict__ dy, float* __restrict__ loss) {
  __shared__ float red[256];
  float s = 0.0f;
  for (int b = threadIdx.x; b < B; b += 256) {
    const float r = y[b] - t[b];
    dy[b] = 2.0f * r / (float)B;
    s = fmaf(r, r, s);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = red[0] / (float)B;
}

// out[j] = sum_b M[b][j] * (wgt ? wgt[b] : 1), j < N. Sixteen slices of the
// workgroup sum rows b = slice, slice + 16, ... in order, then the slices add
// up in order: one thread per column walked B dependent loads (27.7 us for 256
// rows).
constexpr int kSumSlices = 16, kSumCols = 16;
__global__ __launch_bounds__(kSumSlices * kSumCols) void k_colsum(const float* __restrict__ M,
                                                                  const float* __restrict__ wgt, int B, int N,
                                                                  float* __restrict__ out) {
  __shared__ float red[kSumSlices][kSumCols];
  const int c = threadIdx.x % kSumCols, r = threadIdx.x / kSumCols;
  const int j = blockIdx.x * kSumCols + c;
  float s = 0.0f;
  if (j < N)
    for (int b = r; b < B; b += kSumSlices) s = fmaf(M[(long)b * N + j], wgt ? wgt[b] : 1.0f, s);
  red[r][c] = s;
  __syncthreads();
  if (r == 0 && j < N) {
    for (int i = 1; i < kSumSlices; ++i) s += red[i][c];
    out[j] = s;
  }
}

// dz2[b][h] = dy[b] w3[h] (1 - h2[b][h]^2)
__global__ void k_nn_dz2(const float* __restrict__ dy, const float* __restrict__ w3, const float* __restrict__ h2,
                         int B, int H, float* __restrict__ dz2) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)B * H) return;
  const int b = (int)(t / H), h = (int)(t - (long)b * H);
  const float a = h2[t];
  dz2[t] = dy[b] * w3[h] * (1.0f - a * a);
}

// Adam: m = b1 m + (1 - b1) g; v = b2 v + (1 - b2) g^2;
// theta -= lr (m / c1) / (sqrt(v / c2) + eps), c1 = 1 - b1^t, c2 = 1 - b2^t
__device__ __forceinline__ void adam_one(float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v,
                                         long i, float gi, const NNAdam& o) {
  const float mi = o.b1 * m[i] + (1.0f - o.b1) * gi;
  const float vi = o.b2 * v[i] + (1.0f - o.b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  theta[i] -= o.lr * (mi / o.c1) / (sqrtf(vi / o.c2) + o.eps);
}

__global__ void k_adam(float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, long n, NNAdam o) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) adam_one(theta, m, v, i, g[i], o);
}

// training batch from trajectories: for sample s = idx[b] = traj * T + t,
// X[b][w] = seqA[traj][t - W + 1 + w] (0 before the start), target[b] = seqJ[traj][t]
__global__ void k_nn_gather(const float* __restrict__ seqA, const float* __restrict__ seqJ, int T, int W,
                            const int* __restrict__ idx, int B, float* __restrict__ X, float* __restrict__ target) {
  const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (long)B * W) return;
  const int b = (int)(q / W), w = (int)(q - (long)b * W);
  const int s = idx[b];
  const int tr = s / T, t = s - tr * T;
  const int src = t - W + 1 + w;
  X[q] = src >= 0 ? seqA[(long)tr * T + src] : 0.0f;
  if (w == W - 1) target[b] = seqJ[(long)tr * T + t];
}

// dst[0] += src[0]
__global__ void k_accum(const float* __restrict__ src, float* __restrict__ dst) {
  if (threadIdx.x == 0) dst[0] += src[0];
}

// ---------------------------------------------------------------- training step
// One Adam step on a batch in two launches, for hidden widths up to 64,
// windows up to 1024 and batches up to 4096. As seventeen launches (window
// gather, three products, sums, Adam) a batch of 256 with W = 512, H = 16 takes
// 62 us, nearly all launch latency; as two it is 28 us (kernels of 14.5 and
// 6.3 us: dependent loads and eight barriers on 16 workgroups).
// Width: the hidden layers are H products a thread in order, which catches up
// with the launches at 64 (us a batch, seventeen launches / two: W = 512, H = 64,
// B = 256 64 / 51; W = 1024 74 / 69; B = 64 60 / 62). Window and batch: what the
// LDS of the two kernels holds at that width with room to spare (116 of 160 KB,
// 32 KB), not where two launches stop gaining (W = 1024, H = 64, B = 4096
// 401 / 161).
//
// k_nn_tile: sixteen samples per workgroup, forward and backward down to dz1,
// with their windows read from the trajectories into LDS; writes dz1, dy and
// the tile's sums for the small parameters (b1, W2, b2, w3, b3) and the loss.
// k_nn_update: a 16 x 16 tile of W1 per workgroup, gW1 = dz1^T X on the matrix
// cores with the windows again read from the trajectories, then Adam on the
// tile; the last workgroups add up the small parameters' sums in tile order.
constexpr int kFusedH = 64, kFusedW = 1024, kFusedB = 4096;

struct NNTrain {
  const float* seqA;   // [n_traj][T]
  const float* seqJ;
  const int* idx;      // [B] sample = traj * T + t
  int T, B, W, H;
  float *theta, *m, *v, *grad;
  float *dz1, *dy, *part;
  float* loss;         // the batch's mean loss is added to it
  int freeze;          // b3 and ws get a zero gradient
};

__host__ __device__ inline long nn_small(int H) { return (long)H * H + 3L * H + 1; }

bool nn_fused(const NNShape& sh, int B) { return sh.H <= kFusedH && sh.W <= kFusedW && B <= kFusedB; }
// room for any fused batch of at most B samples
size_t nn_part_floats(const NNShape& sh, int B) {
  if (!nn_fused(sh, 1)) return 1;
  return (size_t)((std::min(B, kFusedB) + 15) / 16) * (nn_small(sh.H) + 1);
}

constexpr int kTileWaves = 8, kTileThreads = 64 * kTileWaves;

template <int HT>  // 16-wide tiles of the hidden layer
__global__ __launch_bounds__(kTileThreads) void k_nn_tile(NNTrain a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int HP = 16 * HT, HS = HP + 1;
  const int W = a.W, H = a.H, W16 = (W + 15) / 16 * 16, XS = W16 + 4;
  float* X = reinterpret_cast<float*>(smem_raw);   // [16][XS], zero beyond W
  float* zp = X + 16 * XS;                          // [kTileWaves][16][HS] partial products of the wavefronts
  float* h1 = zp + kTileWaves * 16 * HS;                     // [16][HS] each
  float* h2 = h1 + 16 * HS;
  float* d2 = h2 + 16 * HS;
  float* d1 = d2 + 16 * HS;
  float* sk = d1 + 16 * HS;                         // [16] skip, then dy
  float* rr = sk + 16;                              // [16] squared residuals
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b0 = blockIdx.x * 16;
  const float* W1 = a.theta;
  const float* b1 = W1 + (long)H * W;
  const float* W2 = b1 + H;
  const float* b2 = W2 + (long)H * H;
  const float* w3 = b2 + H;
  const float* b3 = w3 + H;
  const float* ws = b3 + 1;
  // windows: 32 threads per sample
  {
    const int s = tid >> 5;
    const int smp = b0 + s < a.B ? a.idx[b0 + s] : -1;
    const int tr = smp / a.T, t = smp - tr * a.T, lo = t - W + 1;
    const float* q = a.seqA + (long)tr * a.T + lo;
    for (int w = tid & 31; w < W16; w += 32) {
      float x = 0.0f;
      if (smp >= 0 && w < W && lo + w >= 0) x = q[w];
      X[s * XS + w] = x;
    }
  }
  __syncthreads();
  // z1 = X W1^T: each wavefront a contiguous share of the groups of 16 window
  // points; within a group lane (r, q) holds points 4 q .. 4 q + 3. The
  // weights of kAhead groups are loaded before their products.
  const int r = lane & 15, q = lane >> 4;
  const int groups = W16 / 16, per = (groups + kTileWaves - 1) / kTileWaves;
  const int g0 = wave * per, g1 = min(groups, g0 + per);
  constexpr int kAhead = HT <= 2 ? 4 : 2;
  f32x4 acc[HT];
#pragma unroll
  for (int h = 0; h < HT; ++h) acc[h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  for (int gc = g0; gc < g1; gc += kAhead) {
    f32x4 wv[kAhead][HT];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int w0 = 16 * (gc + u) + 4 * q;
#pragma unroll
      for (int h = 0; h < HT; ++h) {
        const float* src = W1 + (long)min(16 * h + r, H - 1) * W;
#pragma unroll
        for (int e = 0; e < 4; ++e) wv[u][h][e] = src[min(w0 + e, W - 1)];
      }
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (gc + u >= g1) break;  // uniform over the wavefront
      const int w0 = 16 * (gc + u) + 4 * q;
      const f32x4 xv = *reinterpret_cast<const f32x4*>(X + r * XS + w0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int h = 0; h < HT; ++h) {
          const float w = 16 * h + r < H && w0 + e < W ? wv[u][h][e] : 0.0f;
          acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[e], w, acc[h], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int h = 0; h < HT; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) zp[(wave * 16 + 4 * q + e) * HS + 16 * h + r] = acc[h][e];
  // the linear skip, two samples per wavefront
  {
    float t0 = 0.0f, t1 = 0.0f;
    const float* x0 = X + 2 * wave * XS;
    for (int w = lane; w < W; w += 64) {
      const float v = ws[w];
      t0 = fmaf(x0[w], v, t0);
      t1 = fmaf(x0[XS + w], v, t1);
    }
    t0 = wave_sum_f(t0);
    t1 = wave_sum_f(t1);
    if (lane == 0) {
      sk[2 * wave] = t0;
      sk[2 * wave + 1] = t1;
    }
  }
  __syncthreads();
  for (int i = tid; i < 16 * H; i += kTileThreads) {
    const int s = i / H, h = i - s * H;
    float z = zp[s * HS + h];
    for (int wv = 1; wv < kTileWaves; ++wv) z += zp[(wv * 16 + s) * HS + h];
    h1[s * HS + h] = tanhf(z + b1[h]);
  }
  __syncthreads();
  for (int i = tid; i < 16 * H; i += kTileThreads) {
    const int s = i / H, h = i - s * H;
    float z = 0.0f;
    for (int k = 0; k < H; ++k) z = fmaf(h1[s * HS + k], W2[(long)h * H + k], z);
    h2[s * HS + h] = tanhf(z + b2[h]);
  }
  __syncthreads();
  if (tid < 256) {
    // y, dy and the residual: sixteen lanes per sample
    const int s = tid >> 4, l = tid & 15;
    float y = 0.0f;
    for (int h = l; h < H; h += 16) y = fmaf(h2[s * HS + h], w3[h], y);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) y += __shfl_xor(y, o, 16);
    if (l == 0) {
      float res = 0.0f;
      if (b0 + s < a.B) res = y + b3[0] + sk[s] - a.seqJ[a.idx[b0 + s]];
      const float dy = 2.0f * res / (float)a.B;
      rr[s] = res * res;
      sk[s] = dy;
      if (b0 + s < a.B) a.dy[b0 + s] = dy;
    }
  }
  __syncthreads();
  for (int i = tid; i < 16 * H; i += kTileThreads) {
    const int s = i / H, h = i - s * H;
    const float v = h2[s * HS + h];
    d2[s * HS + h] = sk[s] * w3[h] * (1.0f - v * v);
  }
  __syncthreads();
  for (int i = tid; i < 16 * H; i += kTileThreads) {
    const int s = i / H, k = i - s * H;
    float z = 0.0f;
    for (int h = 0; h < H; ++h) z = fmaf(d2[s * HS + h], W2[(long)h * H + k], z);
    const float v = h1[s * HS + k];
    z *= 1.0f - v * v;
    d1[s * HS + k] = z;
    if (b0 + s < a.B) a.dz1[(long)(b0 + s) * H + k] = z;
  }
  __syncthreads();
  // the tile's sums for b1, W2, b2, w3, b3 and the loss (samples in order)
  const int ns = (int)nn_small(H);
  float* out = a.part + (long)blockIdx.x * (ns + 1);
  for (int i = tid; i <= ns; i += kTileThreads) {
    float z = 0.0f;
    if (i < H) {
      for (int s = 0; s < 16; ++s) z += d1[s * HS + i];
    } else if (i < H + H * H) {
      const int h = (i - H) / H, k = (i - H) - h * H;
      for (int s = 0; s < 16; ++s) z = fmaf(d2[s * HS + h], h1[s * HS + k], z);
    } else if (i < 2 * H + H * H) {
      for (int s = 0; s < 16; ++s) z += d2[s * HS + i - H - H * H];
    } else if (i < 3 * H + H * H) {
      for (int s = 0; s < 16; ++s) z = fmaf(sk[s], h2[s * HS + i - 2 * H - H * H], z);
    } else if (i == ns - 1) {
      for (int s = 0; s < 16; ++s) z += sk[s];
    } else {
      for (int s = 0; s < 16; ++s) z += rr[s];
    }
    out[i] = z;
  }
}

__global__ __launch_bounds__(256) void k_nn_update(NNTrain a, NNAdam o, int w_tiles, int h_tiles) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ float zp[4][16][17];
  const int W = a.W, H = a.H, B = a.B, tid = threadIdx.x;
  const long oW1 = 0, oSmall = (long)H * W, ns = nn_small(H), oWs = oSmall + ns;
  const int blk = blockIdx.x;
  if (blk >= w_tiles * h_tiles) {
    // small parameters, one per thread: the tiles' sums in order
    const long i = (long)(blk - w_tiles * h_tiles) * 256 + tid;
    if (i > ns) return;
    const int tiles = (B + 15) / 16;
    float g = 0.0f;
    for (int t = 0; t < tiles; ++t) g += a.part[(long)t * (ns + 1) + i];
    if (i == ns) {
      a.loss[0] += g / (float)B;
      return;
    }
    if (i == ns - 1 && a.freeze) g = 0.0f;
    a.grad[oSmall + i] = g;
    adam_one(a.theta, a.m, a.v, oSmall + i, g, o);
    return;
  }
  int* start = reinterpret_cast<int*>(smem_raw);   // [B] first window point in seqA
  int* skip = start + B;                            // [B] window points before the trajectory's start
  for (int b = tid; b < B; b += 256) {
    const int smp = a.idx[b], tr = smp / a.T, t = smp - tr * a.T;
    start[b] = smp - W + 1;
    skip[b] = W - 1 - t;
  }
  __syncthreads();
  const int lane = tid & 63, wave = tid >> 6, r = lane & 15, q = lane >> 4;
  const int w0 = (blk % w_tiles) * 16, h0 = (blk / w_tiles) * 16;
  const int w = w0 + r, h = h0 + r;
  const int steps = (B + 3) / 4, per = (steps + 3) / 4;
  const int s0 = wave * per, s1 = min(steps, s0 + per);
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int kChunk = 8;
  for (int c0 = s0; c0 < s1; c0 += kChunk) {
    float av[kChunk], bv[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const int b = 4 * (c0 + u) + q, bc = min(b, B - 1);
      const bool in = c0 + u < s1 && b < B;
      const bool xin = in && w < W && w >= skip[bc];
      const float dv = a.dz1[(long)bc * H + min(h, H - 1)];
      const float xv = a.seqA[xin ? start[bc] + w : 0];
      av[u] = in && h < H ? dv : 0.0f;
      bv[u] = xin ? xv : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kChunk; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[u], acc, 0, 0, 0);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) zp[wave][4 * q + e][r] = acc[e];
  __syncthreads();
  {
    const int i = tid >> 4, j = tid & 15;
    if (h0 + i < H && w0 + j < W) {
      const float g = zp[0][i][j] + zp[1][i][j] + zp[2][i][j] + zp[3][i][j];
      const long at = oW1 + (long)(h0 + i) * W + w0 + j;
      a.grad[at] = g;
      adam_one(a.theta, a.m, a.v, at, g, o);
    }
  }
  if (h0 > 0) return;
  // the skip weights of these window points: sixteen slices of the batch
  __syncthreads();
  float g = 0.0f;
  const int j = tid & 15, sl = tid >> 4, wj = w0 + j;
  if (!a.freeze && wj < W)
    for (int b = sl; b < B; b += 16)
      if (wj >= skip[b]) g = fmaf(a.dy[b], a.seqA[start[b] + wj], g);
  zp[0][sl][j] = g;
  __syncthreads();
  if (sl == 0 && wj < W) {
    for (int i = 1; i < 16; ++i) g += zp[0][i][j];
    a.grad[oWs + wj] = g;
    adam_one(a.theta, a.m, a.v, oWs + wj, g, o);
  }
}

// ---------------------------------------------------------------- launchers
static hipError_t gemm(const float* A, long sai, long sak, const float* B, long sbk, long sbj, float* C, int M,
                       int N, int K, const float* bias, int act, const float* aux, hipStream_t s) {
  const dim3 grid((unsigned)((N + kTile - 1) / kTile), (unsigned)((M + kTile - 1) / kTile));
  hipLaunchKernelGGL(k_gemm, grid, dim3(kGemmWaves * 64), 0, s, A, sai, sak, B, sbk, sbj, C, M, N, K, bias, act,
                     aux);
  return hipGetLastError();
}

__global__ void k_zero_f(float* __restrict__ p, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

// G[i][i] += lambda_rel * trace(G) / n (one workgroup, fixed-order sum)
__global__ __launch_bounds__(1024) void k_lin_trace_scale(double* __restrict__ G, int n, double lambda_rel,
                                                          int* __restrict__ ok) {
  __shared__ double red[1024];
  const int t = threadIdx.x;
  if (t == 0) *ok = 1;
  double s = 0.0;
  for (int i = t; i < n; i += 1024) s += G[(size_t)i * n + i];
  red[t] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  const double lam = lambda_rel * red[0] / n;
  __syncthreads();
  for (int i = t; i < n; i += 1024) G[(size_t)i * n + i] += lam;
}

// ---------------------------------------------------------------------------
// Least-squares fit of the linear part (skip weights and output bias) over a
// set of trajectories, FP64. With the regressors x = (window of A, 1), n = W + 1:
//   G[i][j] = sum over samples of x_i x_j,  b[i] = sum x_i y,
// then (G + lambda I) w = b by a Cholesky factorisation.
// Window entry i of the sample at time t of a trajectory is A(t - W + 1 + i),
// zero before t = 0.

// The windows of a trajectory are shifts of one series, so the matrix is summed
// along its diagonals: with d = j - i and a(s) the series,
//   G[i][i + d] = sum over trajectories of sum_{s = 0}^{T - W + i} a(s) a(s + d),
// a running sum over s per lag d (W T products per trajectory; pair by pair it
// is W^2 T / 2 of them, 2.4 ms for W = 512 and 13200 samples). One workgroup
// per lag; d = W: the column of the constant, with a(s) alone. Only the lower
// triangle G[i + d][i] is written; row n of G is the right-hand side.
__device__ __forceinline__ void lin_lag(const double* __restrict__ A, int n_traj, int T, int W,
                                        double* __restrict__ G, int d, double (&sc)[256]) {
  const int n = W + 1, tid = threadIdx.x;
  const bool one = d == W;
  const int cnt = one ? W : W - d;      // entries i = 0 .. cnt - 1
  const int shift = T - W;              // entry i is the running sum at s = shift + i
  auto put = [&](int i, double v) { G[one ? (size_t)W * n + i : (size_t)(i + d) * n + i] = v; };
  for (int i = tid; i < min(cnt, -shift); i += 256) put(i, 0.0);  // windows that never reach the series
  double carry = 0.0;
  const int smax = shift + cnt - 1;     // <= T - 1 - d
  for (int s0 = 0; s0 <= smax; s0 += 256) {
    const int s = s0 + tid;
    double c = 0.0;
    if (s <= smax)
      for (int k = 0; k < n_traj; ++k) {
        const double* a = A + (size_t)k * T;
        c += one ? a[s] : a[s] * a[s + d];
      }
    sc[tid] = c;
    __syncthreads();
    for (int h = 1; h < 256; h <<= 1) {
      const double v = tid >= h ? sc[tid - h] : 0.0;
      __syncthreads();
      sc[tid] += v;
      __syncthreads();
    }
    if (s <= smax && s >= shift) put(s - shift, carry + sc[tid]);
    carry += sc[255];
    __syncthreads();
  }
  if (one && tid == 0) G[(size_t)W * n + W] = (double)n_traj * T;
}

// the right-hand side b[i] = sum x_i y (row n of G): one workgroup per entry,
// thread t sums samples t, t + 256, ... in order, then a fixed pairwise tree
__device__ __forceinline__ void lin_rhs(const double* __restrict__ A, const double* __restrict__ Y, int n_traj, int T,
                                        int W, double* __restrict__ G, int i, double (&red)[256]) {
  const int n = W + 1, tid = threadIdx.x;
  const int t0 = i == W ? 0 : max(0, W - 1 - i);  // first sample whose window entry i is inside
  double acc = 0.0;
  for (int k = 0; k < n_traj; ++k)
    for (int t = t0 + tid; t < T; t += 256) {
      const double y = Y[(size_t)k * T + t];
      acc += i == W ? y : y * A[(size_t)k * T + t - W + 1 + i];
    }
  red[tid] = acc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  if (tid == 0) G[(size_t)n * n + i] = red[0];
}

// the lags by workgroups 0 .. W, the right-hand side by W + 1 .. 2 W + 1
__global__ __launch_bounds__(256) void k_lin_sums(const double* __restrict__ A, const double* __restrict__ Y,
                                                  int n_traj, int T, int W, double* __restrict__ G) {
  __shared__ double buf[256];
  const int b = blockIdx.x;
  if (b <= W)
    lin_lag(A, n_traj, T, W, G, b, buf);
  else
    lin_rhs(A, Y, n_traj, T, W, G, b - W - 1, buf);
}

// Cholesky G = L L^T by panels of kPanel columns, rows 0 .. n (the last is the
// right-hand side, whose row of L is the forward substitution's result), then
// the back substitution. In one workgroup, column by column, the 513 columns
// of a 512-point window took 15.9 ms; by panels 0.55 ms (17 panels of 19 us,
// 16 updates of 6 us and the back substitution 0.13 ms, all latency).
constexpr int kPanel = 32;

__device__ __forceinline__ double lane_read(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// The panel at column j: every workgroup factors the diagonal block (kept in
// Ld, so that G's is not overwritten while others read it) and solves 64 rows
// below it. *ok = 0 if a pivot is not positive. A matrix of one panel (one
// workgroup then) gets its lambda here, by k_lin_trace_scale's tree: with that
// launch, one of its own for the right-hand side and padded columns factored
// too, a call with a window of one sample took 85 us (everything in one
// workgroup 75), now 73; a window of 64 is 136 -> 125 us.
// PART: the last columns, fewer than a panel's (that test in a full panel's
// code costs a window of 64 its gain).
template <bool PART>
__global__ __launch_bounds__(64) void k_chol_panel(double* __restrict__ G, double* __restrict__ Ld, int n, int j,
                                                   double lambda_rel, int* __restrict__ ok) {
  __shared__ double D[kPanel][kPanel + 1];
  const int lane = threadIdx.x, nb = PART ? n - j : kPanel;
  for (int i = lane; i < kPanel * kPanel; i += 64) {
    const int r = i / kPanel, c = i % kPanel;
    D[r][c] = r < nb && c <= r ? G[(size_t)(j + r) * n + j + c] : (r == c ? 1.0 : 0.0);
  }
  __syncthreads();
  if (n <= kPanel) {
    double s = lane < n ? D[lane][lane] : 0.0;
#pragma unroll
    for (int h = kPanel / 2; h > 0; h >>= 1) s += __shfl_xor(s, h, 64);
    if (lane < n) D[lane][lane] += lambda_rel * s / n;
    if (lane == 0) *ok = 1;
    __syncthreads();
  }
  // the block's row lane & 31 in registers; the values of other rows come by
  // lane reads
  const int r = lane & 31;
  double a[kPanel];
#pragma unroll
  for (int c = 0; c < kPanel; ++c) a[c] = D[r][c];
  bool good = true;
#pragma unroll
  for (int c = 0; c < kPanel; ++c) {
    if (PART && c >= nb) continue;  // uniform; the padding is its own factor
    double d = lane_read(a[c], c);
    if (!(d > 0.0)) {
      good = false;
      d = 1.0;
    }
    const double piv = sqrt(d);
    a[c] = r == c ? piv : a[c] / piv;
#pragma unroll
    for (int k = c + 1; k < kPanel; ++k) {
      a[k] -= a[c] * lane_read(a[c], k);  // of use where k <= r
      // keeps the lane reads (scalar registers) next to their use
      if (k % 16 == 15) __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (!good && blockIdx.x == 0 && lane == 0) *ok = 0;
  __syncthreads();
  if (lane < kPanel) {
#pragma unroll
    for (int c = 0; c < kPanel; ++c) D[r][c] = c <= r ? a[c] : 0.0;
  }
  __syncthreads();
  if (blockIdx.x == 0)
    for (int i = lane; i < kPanel * kPanel; i += 64)
      Ld[(size_t)(j / kPanel) * kPanel * kPanel + i] = D[i / kPanel][i % kPanel];
  const int row = j + kPanel + blockIdx.x * 64 + lane;
  if (PART) {
    // only the right-hand side (row n) is left below it
    if (blockIdx.x > 0 || lane > 0) return;
    for (int c = 0; c < nb; ++c) {
      double x = G[(size_t)n * n + j + c];
      for (int k = 0; k < c; ++k) x -= G[(size_t)n * n + j + k] * D[c][k];
      G[(size_t)n * n + j + c] = x / D[c][c];
    }
    return;
  }
  if (row > n) return;
  double x[kPanel];
#pragma unroll
  for (int c = 0; c < kPanel; ++c) x[c] = G[(size_t)row * n + j + c];
#pragma unroll
  for (int c = 0; c < kPanel; ++c) {
#pragma unroll
    for (int k = 0; k < c; ++k) x[c] -= x[k] * D[c][k];
    x[c] /= D[c][c];
  }
#pragma unroll
  for (int c = 0; c < kPanel; ++c) G[(size_t)row * n + j + c] = x[c];
}

// G[r][c] -= sum_k L[r][j + k] L[c][j + k] for the 32 x 32 tile (blockIdx.y,
// blockIdx.x) below and right of the panel at j (lower tiles only)
__global__ __launch_bounds__(256) void k_chol_update(double* __restrict__ G, int n, int j) {
  if (blockIdx.x > blockIdx.y) return;
  __shared__ double R[32][kPanel + 1], C[32][kPanel + 1];
  const int r0 = j + kPanel + blockIdx.y * 32, c0 = j + kPanel + blockIdx.x * 32, tid = threadIdx.x;
  for (int i = tid; i < 32 * kPanel; i += 256) {
    const int a = i / kPanel, k = i % kPanel;
    R[a][k] = r0 + a <= n ? G[(size_t)(r0 + a) * n + j + k] : 0.0;
    C[a][k] = c0 + a < n ? G[(size_t)(c0 + a) * n + j + k] : 0.0;
  }
  __syncthreads();
  const int c = tid & 31;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int a = (tid >> 5) + 8 * u;
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kPanel; ++k) acc += R[a][k] * C[c][k];
    if (r0 + a <= n && c0 + c < n && c0 + c <= r0 + a) G[(size_t)(r0 + a) * n + c0 + c] -= acc;
  }
}

// L^T w = z with z in row n of G (overwritten): blocks from the last, the
// triangle by one wavefront, the rest by the workgroup
__global__ __launch_bounds__(1024) void k_chol_back(double* __restrict__ G, const double* __restrict__ Ld, int n,
                                                    float* __restrict__ ws, float* __restrict__ b3) {
  __shared__ double w[kPanel];
  double* z = G + (size_t)n * n;
  const int tid = threadIdx.x;
  for (int j = (n - 1) / kPanel * kPanel; j >= 0; j -= kPanel) {
    const int nb = min(kPanel, n - j);
    if (tid < 64) {
      // lane k holds column k of the block (padded with the identity)
      const double* D = Ld + (size_t)(j / kPanel) * kPanel * kPanel;
      const int k = tid & 31;
      double d[kPanel];
#pragma unroll
      for (int c = 0; c < kPanel; ++c) d[c] = D[c * kPanel + k];
      double x = k < nb ? z[j + k] : 0.0;
#pragma unroll
      for (int c = kPanel - 1; c >= 0; --c) {
        if (c >= nb) continue;
        const double wc = lane_read(x, c) / lane_read(d[c], c);
        if (k == c) x = wc;
        if (k < c) x -= d[c] * wc;
      }
      if (tid < kPanel) w[tid] = x;
      if (tid < nb) z[j + tid] = x;
    }
    __syncthreads();
    for (int i = tid; i < j; i += 1024) {
      double acc = z[i];
#pragma unroll 16
      for (int c = 0; c < kPanel; ++c)
        if (c < nb) acc -= G[(size_t)(j + c) * n + i] * w[c];
      z[i] = acc;
    }
    __syncthreads();
  }
  for (int i = tid; i < n - 1; i += 1024) ws[i] = (float)z[i];
  if (tid == 0) *b3 = (float)z[n - 1];
}

size_t nn_fit_doubles(int W) {
  const size_t n = (size_t)W + 1;
  return (n + 1) * n + (n + kPanel - 1) / kPanel * kPanel * kPanel;
}

hipError_t nn_fit_linear(const double* A, const double* Y, int n_traj, int T, int W, double lambda_rel, double* G,
                         float* ws, float* b3, int* ok, hipStream_t s) {
  const int n = W + 1;
  double* Ld = G + (size_t)(n + 1) * n;
  hipLaunchKernelGGL(k_lin_sums, dim3((unsigned)(2 * n)), dim3(256), 0, s, A, Y, n_traj, T, W, G);
  // lambda relative to the mean diagonal of G
  if (n > kPanel) hipLaunchKernelGGL(k_lin_trace_scale, dim3(1), dim3(1024), 0, s, G, n, lambda_rel, ok);
  for (int j = 0; j < n; j += kPanel) {
    const int below = n + 1 - j - kPanel;  // rows under the panel, the right-hand side among them
    const dim3 grid((unsigned)max(1, (below + 63) / 64));
    if (n - j < kPanel)
      hipLaunchKernelGGL(k_chol_panel<true>, grid, dim3(64), 0, s, G, Ld, n, j, lambda_rel, ok);
    else
      hipLaunchKernelGGL(k_chol_panel<false>, grid, dim3(64), 0, s, G, Ld, n, j, lambda_rel, ok);
    if (below > 0) {
      const unsigned tr = (unsigned)((below + 31) / 32), tc = (unsigned)((n - j - kPanel + 31) / 32);
      if (tc > 0) hipLaunchKernelGGL(k_chol_update, dim3(tc, tr), dim3(256), 0, s, G, n, j);
    }
  }
  hipLaunchKernelGGL(k_chol_back, dim3(1), dim3(1024), 0, s, G, Ld, n, ws, b3);
  return hipGetLastError();
}

hipError_t nn_zero(float* p, long n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_f, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t nn_forward(const NNShape& sh, const float* theta, const float* X, int B, NNWork& wk, hipStream_t s) {
  const int W = sh.W, H = sh.H;
  const float* W1 = theta;
  const float* b1 = W1 + (long)H * W;
  const float* W2 = b1 + H;
  const float* b2 = W2 + (long)H * H;
  const float* w3 = b2 + H;
  const float* b3 = w3 + H;
  const float* ws = b3 + 1;
  hipError_t e;
  // h1 = tanh(X W1^T + b1): A = X [B][W], B(k=w, j=h) = W1[h][w]
  if ((e = gemm(X, W, 1, W1, 1, W, wk.h1, B, H, W, b1, 1, nullptr, s)) != hipSuccess) return e;
  if ((e = gemm(wk.h1, H, 1, W2, 1, H, wk.h2, B, H, H, b2, 1, nullptr, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_nn_out, dim3((unsigned)((B + 3) / 4)), dim3(256), 0, s, wk.h2, X, w3, b3, ws, B, H, W, wk.y);
  return hipGetLastError();
}

static void colsum(const float* M, const float* wgt, int B, int N, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_colsum, dim3((unsigned)((N + kSumCols - 1) / kSumCols)), dim3(kSumSlices * kSumCols), 0, s, M,
                     wgt, B, N, out);
}

hipError_t nn_backward(const NNShape& sh, const float* theta, const float* X, const float* target, int B,
                       NNWork& wk, float* grad, hipStream_t s) {
  const int W = sh.W, H = sh.H;
  const float* W2 = theta + (long)H * W + H;
  const float* w3 = W2 + (long)H * H + H;
  float* gW1 = grad;
  float* gb1 = gW1 + (long)H * W;
  float* gW2 = gb1 + H;
  float* gb2 = gW2 + (long)H * H;
  float* gw3 = gb2 + H;
  float* gb3 = gw3 + H;
  float* gws = gb3 + 1;
  hipError_t e;
  hipLaunchKernelGGL(k_nn_dy_loss, dim3(1), dim3(256), 0, s, wk.y, target, B, wk.dy, wk.loss);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  colsum(wk.h2, wk.dy, B, H, gw3, s);
  colsum(wk.dy, nullptr, B, 1, gb3, s);
  colsum(X, wk.dy, B, W, gws, s);
  hipLaunchKernelGGL(k_nn_dz2, dim3((unsigned)(((long)B * H + 255) / 256)), dim3(256), 0, s, wk.dy, w3, wk.h2, B,
                     H, wk.dz2);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // gW2[h][k] = sum_b dz2[b][h] h1[b][k]: A(i=h, k=b) = dz2[b][h], B(k=b, j) = h1[b][j]
  if ((e = gemm(wk.dz2, 1, H, wk.h1, H, 1, gW2, H, H, B, nullptr, 0, nullptr, s)) != hipSuccess) return e;
  colsum(wk.dz2, nullptr, B, H, gb2, s);
  // dz1[b][k] = (sum_h dz2[b][h] W2[h][k]) (1 - h1[b][k]^2)
  if ((e = gemm(wk.dz2, H, 1, W2, H, 1, wk.dz1, B, H, H, nullptr, 0, wk.h1, s)) != hipSuccess) return e;
  // gW1[h][w] = sum_b dz1[b][h] X[b][w]
  if ((e = gemm(wk.dz1, 1, H, X, W, 1, gW1, H, W, B, nullptr, 0, nullptr, s)) != hipSuccess) return e;
  colsum(wk.dz1, nullptr, B, H, gb1, s);
  return hipGetLastError();
}

hipError_t nn_adam(float* theta, float* m, float* v, const float* g, long n, const NNAdam& o, hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, theta, m, v, g, n, o);
  return hipGetLastError();
}

hipError_t nn_gather(const float* seqA, const float* seqJ, int T, int W, const int* idx, int B, float* X,
                     float* target, hipStream_t s) {
  const long n = (long)B * W;
  hipLaunchKernelGGL(k_nn_gather, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, seqA, seqJ, T, W, idx, B, X,
                     target);
  return hipGetLastError();
}

hipError_t nn_accumulate(const float* src, float* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_accum, dim3(1), dim3(64), 0, s, src, dst);
  return hipGetLastError();
}

hipError_t nn_train_step(const NNShape& sh, float* theta, float* m, float* v, float* grad, const float* seqA,
                         const float* seqJ, int T, const int* idx, int B, NNWork& wk, const NNAdam& o, int freeze,
                         float* loss, hipStream_t s) {
  if (!nn_fused(sh, B) || B < 1) return hipErrorInvalidValue;
  const NNTrain a{seqA, seqJ, idx, T, B, sh.W, sh.H, theta, m, v, grad, wk.dz1, wk.dy, wk.part, loss, freeze};
  const int HT = (sh.H + 15) / 16, HS = 16 * HT + 1, XS = (sh.W + 15) / 16 * 16 + 4;
  const size_t lds = ((size_t)16 * XS + (kTileWaves + 4) * 16 * HS + 32) * sizeof(float);
  const dim3 grid((unsigned)((B + 15) / 16));
  switch (HT) {
    case 1: hipLaunchKernelGGL(k_nn_tile<1>, grid, dim3(kTileThreads), lds, s, a); break;
    case 2: hipLaunchKernelGGL(k_nn_tile<2>, grid, dim3(kTileThreads), lds, s, a); break;
    case 3: hipLaunchKernelGGL(k_nn_tile<3>, grid, dim3(kTileThreads), lds, s, a); break;
    default: hipLaunchKernelGGL(k_nn_tile<4>, grid, dim3(kTileThreads), lds, s, a); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int wt = (sh.W + 15) / 16, sm = (int)((nn_small(sh.H) + 1 + 255) / 256);
  hipLaunchKernelGGL(k_nn_update, dim3((unsigned)(wt * HT + sm)), dim3(256), (size_t)2 * B * sizeof(int), s, a, o, wt,
                     HT);
  return hipGetLastError();
}

}  // namespace td
