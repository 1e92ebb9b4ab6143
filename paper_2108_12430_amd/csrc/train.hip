// Training-step kernels for the DeepClean-shaped network: batch-statistics
// normalisation (forward and backward, fused with tanh and its derivative),
// per-channel reductions, deterministic weight gradients, and the band-passed
// MSE loss.  Every reduction has a fixed combination order (chunk partials in
// FP64, then a fixed tree), so results are bitwise reproducible and do not
// depend on scheduling.
#include "internal.h"

#include <algorithm>
#include <initializer_list>

namespace gw {

static constexpr int RCHUNK = 4096;  // (batch, time) elements per reduction chunk

// Fixed-order block reduction of two doubles over 256 lanes.
__device__ __forceinline__ void block_sum2(double& a, double& b) {
  __shared__ double sa[256], sb[256];
  sa[threadIdx.x] = a;
  sb[threadIdx.x] = b;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      sa[threadIdx.x] += sa[threadIdx.x + w];
      sb[threadIdx.x] += sb[threadIdx.x + w];
    }
    __syncthreads();
  }
  a = sa[0];
  b = sb[0];
  __syncthreads();
}

enum RMode { R_STATS = 0, R_BNBWD = 1, R_SUM = 2 };

struct RedP {
  const float* x;       // z (stats), g (bnbwd), x (sum): [n][C][L]
  const float* a;       // tanh output (bnbwd)
  const float* z;       // pre-normalisation values (bnbwd)
  const float* mean;
  const float* invstd;
  int n, C, L, nchunk;
  double* partial;      // [C][nchunk][2]
};

// Stage 1: chunk partials.  R_STATS sums (z, z^2); R_BNBWD sums (dh, dh*xhat)
// with dh = g (1 - a^2) and xhat = (z - mean) invstd; R_SUM sums (x, 0).
template <int MODE>
__global__ __launch_bounds__(256) void chan_partial(RedP p) {
  const int q = blockIdx.x, c = blockIdx.y;
  const int64_t N = (int64_t)p.n * p.L;
  double s0 = 0.0, s1 = 0.0;
  float mu = 0.f, is = 0.f;
  if (MODE == R_BNBWD) {
    mu = p.mean[c];
    is = p.invstd[c];
  }
  // this thread's elements e = q RCHUNK + 256 r + tid, (b, t) = (e / L, e % L)
  // tracked incrementally; all loads are issued before the in-order sums
  constexpr int NR = RCHUNK / 256;
  const int64_t e0 = (int64_t)q * RCHUNK + threadIdx.x;
  const int nr = (int)std::max<int64_t>(0, std::min<int64_t>(NR, (N - e0 + 255) / 256));
  int64_t b = e0 / p.L;
  int t = (int)(e0 - b * p.L);
  int64_t idx[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    idx[r] = r < nr ? (b * p.C + c) * p.L + t : 0;
    t += 256;
    while (t >= p.L) {
      t -= p.L;
      ++b;
    }
  }
  float xv[NR], av[MODE == R_BNBWD ? NR : 1], zv[MODE == R_BNBWD ? NR : 1];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    xv[r] = p.x[idx[r]];
    if (MODE == R_BNBWD) {
      av[r] = p.a[idx[r]];
      zv[r] = p.z[idx[r]];
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (r >= nr) break;
    if (MODE == R_STATS) {
      const double v = xv[r];
      s0 += v;
      s1 += v * v;
    } else if (MODE == R_BNBWD) {
      const float dh = xv[r] * (1.0f - av[r] * av[r]);
      const float xh = (zv[r] - mu) * is;
      s0 += (double)dh;
      s1 += (double)dh * (double)xh;
    } else {
      s0 += (double)xv[r];
    }
  }
  block_sum2(s0, s1);
  if (threadIdx.x == 0) {
    p.partial[((int64_t)c * p.nchunk + q) * 2 + 0] = s0;
    p.partial[((int64_t)c * p.nchunk + q) * 2 + 1] = s1;
  }
}

// Stage 2: one block per channel combines the chunk partials in a fixed tree:
// a thread's, a wave's by lane exchange, the waves' in order.  Bound by latency
// (the launch, one round trip to memory, the tree), so all of a thread's loads
// go out at once and the tree has one barrier.
// Outputs (by mode):
//   R_STATS: o0 = mean, o1 = 1/sqrt(var + eps) (biased variance)
//   R_BNBWD: o0 = dbeta = sum dh, o1 = dgamma = sum dh*xhat
//   R_SUM:   o0 = sum
template <int MODE>
__global__ __launch_bounds__(512) void chan_final(const double* partial, int nchunk, int64_t N,
                                                  float* o0, float* o1) {
  const int c = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double2* src = reinterpret_cast<const double2*>(partial) + (int64_t)c * nchunk;
  double s0 = 0.0, s1 = 0.0;
  for (int q = threadIdx.x; q < nchunk; q += 512 * 8) {
    double2 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = q + 512 * j;
      v[j] = src[e < nchunk ? e : nchunk - 1];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (q + 512 * j < nchunk) {
        s0 += v[j].x;
        s1 += v[j].y;
      }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_down(s0, off, 64);
    s1 += __shfl_down(s1, off, 64);
  }
  __shared__ double2 sw[8];
  if (lane == 0) sw[wave] = make_double2(s0, s1);
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int w = 1; w < 8; ++w) {
    s0 += sw[w].x;
    s1 += sw[w].y;
  }
  if (MODE == R_STATS) {
    const double m = s0 / (double)N;
    double v = s1 / (double)N - m * m;
    if (v < 0.0) v = 0.0;
    o0[c] = (float)m;
    o1[c] = (float)(1.0 / sqrt(v + 1e-5));
  } else if (MODE == R_BNBWD) {
    o0[c] = (float)s0;
    o1[c] = (float)s1;
  } else {
    o0[c] = (float)s0;
  }
}

int red_chunks(int n, int L) { return (int)(((int64_t)n * L + RCHUNK - 1) / RCHUNK); }

hipError_t launch_bn_stats(const float* z, int n, int C, int L, double* partial, int nchunk,
                           float* mean, float* invstd, hipStream_t st) {
  RedP p{};
  p.x = z;
  p.n = n;
  p.C = C;
  p.L = L;
  p.nchunk = nchunk;
  p.partial = partial;
  hipLaunchKernelGGL(chan_partial<R_STATS>, dim3(nchunk, C), dim3(256), 0, st, p);
  hipLaunchKernelGGL(chan_final<R_STATS>, dim3(C), dim3(512), 0, st, partial, nchunk,
                     (int64_t)n * L, mean, invstd);
  return hipGetLastError();
}

hipError_t launch_stats_final(const double* partial, int nblk, int C, int64_t N, float* mean, float* invstd,
                              hipStream_t st) {
  hipLaunchKernelGGL(chan_final<R_STATS>, dim3(C), dim3(512), 0, st, partial, nblk, N, mean, invstd);
  return hipGetLastError();
}

hipError_t launch_bnbwd_final(const double* partial, int nblk, int C, int64_t N, float* dgamma, float* dbeta,
                              hipStream_t st) {
  hipLaunchKernelGGL(chan_final<R_BNBWD>, dim3(C), dim3(512), 0, st, partial, nblk, N, dbeta, dgamma);
  return hipGetLastError();
}

hipError_t launch_channel_sum(const float* x, int n, int C, int L, double* partial, int nchunk,
                              float* out, hipStream_t st) {
  RedP p{};
  p.x = x;
  p.n = n;
  p.C = C;
  p.L = L;
  p.nchunk = nchunk;
  p.partial = partial;
  hipLaunchKernelGGL(chan_partial<R_SUM>, dim3(nchunk, C), dim3(256), 0, st, p);
  hipLaunchKernelGGL(chan_final<R_SUM>, dim3(C), dim3(512), 0, st, partial, nchunk,
                     (int64_t)n * L, out, (float*)nullptr);
  return hipGetLastError();
}

// Elementwise kernels over [n][C][L]: grid y = rows (b C + c, strided by
// gridDim.y), x = runs of 1024 positions; 4 positions per thread, as one
// float4 when every row starts 16-byte aligned.
static inline bool rows_vec4(int L, std::initializer_list<const void*> ptrs) {
  if (L % 4) return false;
  for (const void* q : ptrs)
    if (reinterpret_cast<uintptr_t>(q) % 16) return false;
  return true;
}

static inline dim3 rows_grid(int n, int C, int L) {
  const int64_t rows = (int64_t)n * C;
  return dim3((unsigned)((L + 1023) / 1024), (unsigned)std::min<int64_t>(rows, 65535));
}

// a = tanh(gamma (z - mean) invstd + beta)
template <bool V4>
__global__ __launch_bounds__(256) void bn_apply_tanh_kernel(const float* z, const float* mean,
                                                            const float* invstd, const float* gamma,
                                                            const float* beta, float* a, int C,
                                                            int L, int64_t rows) {
  const int t = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (t >= L) return;
  for (int64_t row = blockIdx.y; row < rows; row += gridDim.y) {
    const int c = (int)(row % C);
    const float m = mean[c], is = invstd[c], g = gamma[c], be = beta[c];
    const float* zr = z + row * L + t;
    float* ar = a + row * L + t;
    if (V4) {
      const float4 v = *reinterpret_cast<const float4*>(zr);
      float4 r;
      r.x = tanhf(fmaf(g, (v.x - m) * is, be));
      r.y = tanhf(fmaf(g, (v.y - m) * is, be));
      r.z = tanhf(fmaf(g, (v.z - m) * is, be));
      r.w = tanhf(fmaf(g, (v.w - m) * is, be));
      *reinterpret_cast<float4*>(ar) = r;
    } else {
      for (int j = 0; j < 4 && t + j < L; ++j) ar[j] = tanhf(fmaf(g, (zr[j] - m) * is, be));
    }
  }
}

hipError_t launch_bn_apply_tanh(const float* z, const float* mean, const float* invstd,
                                const float* gamma, const float* beta, float* a, int n, int C,
                                int L, hipStream_t st) {
  const int64_t rows = (int64_t)n * C;
  if (rows < 1 || L < 1) return hipSuccess;
  if (rows_vec4(L, {z, a}))
    hipLaunchKernelGGL(bn_apply_tanh_kernel<true>, rows_grid(n, C, L), dim3(256), 0, st, z, mean, invstd, gamma,
                       beta, a, C, L, rows);
  else
    hipLaunchKernelGGL(bn_apply_tanh_kernel<false>, rows_grid(n, C, L), dim3(256), 0, st, z, mean, invstd, gamma,
                       beta, a, C, L, rows);
  return hipGetLastError();
}

// dz = gamma invstd (dh - sum(dh)/N - xhat sum(dh xhat)/N), dh = g (1 - a^2)
__device__ __forceinline__ float bn_tanh_bwd_one(float g, float av, float zv, float m, float is, float gis,
                                                 float s1, float s2) {
  const float dh = g * (1.0f - av * av);
  const float xh = (zv - m) * is;
  return gis * (dh - s1 - xh * s2);
}

template <bool V4>
__global__ __launch_bounds__(256) void bn_tanh_bwd_kernel(const float* g, const float* a,
                                                          const float* z, const float* mean,
                                                          const float* invstd, const float* gamma,
                                                          const float* sdh, const float* sdhx,
                                                          float* dz, int C, int L, int64_t rows,
                                                          float invN) {
  const int t = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (t >= L) return;
  for (int64_t row = blockIdx.y; row < rows; row += gridDim.y) {
    const int c = (int)(row % C);
    const float m = mean[c], is = invstd[c], gis = gamma[c] * invstd[c];
    const float s1 = sdh[c] * invN, s2 = sdhx[c] * invN;
    const int64_t o = row * L + t;
    if (V4) {
      const float4 gv = *reinterpret_cast<const float4*>(g + o);
      const float4 av = *reinterpret_cast<const float4*>(a + o);
      const float4 zv = *reinterpret_cast<const float4*>(z + o);
      float4 r;
      r.x = bn_tanh_bwd_one(gv.x, av.x, zv.x, m, is, gis, s1, s2);
      r.y = bn_tanh_bwd_one(gv.y, av.y, zv.y, m, is, gis, s1, s2);
      r.z = bn_tanh_bwd_one(gv.z, av.z, zv.z, m, is, gis, s1, s2);
      r.w = bn_tanh_bwd_one(gv.w, av.w, zv.w, m, is, gis, s1, s2);
      *reinterpret_cast<float4*>(dz + o) = r;
    } else {
      for (int j = 0; j < 4 && t + j < L; ++j)
        dz[o + j] = bn_tanh_bwd_one(g[o + j], a[o + j], z[o + j], m, is, gis, s1, s2);
    }
  }
}

hipError_t launch_bn_tanh_backward(const float* g, const float* a, const float* z,
                                   const float* mean, const float* invstd, const float* gamma,
                                   int n, int C, int L, double* partial, int nchunk, float* dz,
                                   float* dgamma, float* dbeta, hipStream_t st) {
  RedP p{};
  p.x = g;
  p.a = a;
  p.z = z;
  p.mean = mean;
  p.invstd = invstd;
  p.n = n;
  p.C = C;
  p.L = L;
  p.nchunk = nchunk;
  p.partial = partial;
  hipLaunchKernelGGL(chan_partial<R_BNBWD>, dim3(nchunk, C), dim3(256), 0, st, p);
  hipLaunchKernelGGL(chan_final<R_BNBWD>, dim3(C), dim3(512), 0, st, partial, nchunk,
                     (int64_t)n * L, dbeta, dgamma);
  const int64_t rows = (int64_t)n * C;
  const float invN = (float)(1.0 / ((double)n * L));
  if (rows_vec4(L, {g, a, z, dz}))
    hipLaunchKernelGGL(bn_tanh_bwd_kernel<true>, rows_grid(n, C, L), dim3(256), 0, st, g, a, z, mean, invstd, gamma,
                       dbeta, dgamma, dz, C, L, rows, invN);
  else
    hipLaunchKernelGGL(bn_tanh_bwd_kernel<false>, rows_grid(n, C, L), dim3(256), 0, st, g, a, z, mean, invstd, gamma,
                       dbeta, dgamma, dz, C, L, rows, invN);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Weight gradient: dw[a][c][j] = sum_b sum_t P[b][a][t] * Q[b][c][s t - p + j]
// (Q zero outside [0, Lq)).  For a conv layer P = dL/dz (a = out channel) and
// Q = layer input; for a transposed layer P = layer input and Q = dL/dz.
// Stage 1, a split-K GEMM on the matrix cores: D[a][n] (n = c k + j) summed
// over K = (batch item, time).  Block g walks a fixed run of chunks (batch
// item, WT time steps) in order.  Each thread loads its share of a chunk (P
// rows and the matching window of Q) into registers in one batch of
// independent loads, and the next chunk's loads are issued before the current
// chunk's MFMAs, so memory latency overlaps compute.  The staged chunk sits in
// LDS (FP32) and v_mfma_f32_16x16x4_f32 (exact FP32 products, FP32
// accumulation) runs over WT / 4 K steps of 4 time steps.  Layers with fewer
// accumulator tiles than waves split each chunk's K steps between wave
// groups, whose accumulators are added in a fixed order at the end.  The
// block's sums are written once as block g's FP32 partial.  Stages 2 and 3 add
// the partials of every weight in a fixed two-level tree (groups of 64
// partials, then the groups) in FP64.  Every order is fixed: the result is
// deterministic.
// ---------------------------------------------------------------------------
static constexpr int WG = 64;    // partials per group of the reduction tree
static constexpr int WNW = 8;    // waves per block
static constexpr int WTH = 64 * WNW;
static constexpr int WTPW = 7;   // most accumulator tiles per wave

// chunk configurations, largest chunk first: time steps, the most P and Q
// elements one thread stages per chunk, the most accumulator tiles per wave
struct WgCfg {
  int wt, pmax, qmax, ntmax;
};
static constexpr WgCfg kWgCfg[] = {{1024, 8, 24, 3}, {512, 8, 24, 3}, {256, 8, 24, 3},
                                   {128, 8, 12, 3},  {64, 8, 12, 7},  {64, 16, 24, 7}};

static int wgrad_qs(int span) { return span + ((16 - span % 64) + 64) % 64; }  // row stride = 16 mod 64 banks

static size_t wgrad_lds(int Ca, int Cc, int k, int s, int wt) {
  const size_t need = sizeof(float) * ((size_t)(Ca + 1) * (wt + 4) + (size_t)(Cc + 1) * wgrad_qs(s * (wt - 1) + k) + WTH);
  return std::max(need, sizeof(float) * 8 * 256);  // room to combine the wave groups' accumulators
}

// wave groups splitting a chunk's K steps: as many as the idle waves allow
// (ntile accumulator tiles, ksp * ntile <= 8 when ntile < 8)
__host__ __device__ inline int wgrad_ksp(int ntile) {
  return ntile >= WNW ? 1 : (2 * ntile > WNW ? 1 : (4 * ntile > WNW ? 2 : (8 * ntile > WNW ? 4 : 8)));
}

// the configuration a layer runs with (index into kWgCfg), -1 if none fits
static int wgrad_cfg(int Ca, int Cc, int k, int s) {
  const int ntile = ((Ca + 15) / 16) * ((Cc * k + 15) / 16);
  const int nwk = WNW / wgrad_ksp(ntile), tpw = (ntile + nwk - 1) / nwk;
  for (int i = 0; i < (int)(sizeof(kWgCfg) / sizeof(kWgCfg[0])); ++i) {
    const WgCfg c = kWgCfg[i];
    const int span = s * (c.wt - 1) + k;
    if (Ca * c.wt <= WTH * c.pmax && Cc * span <= WTH * c.qmax && span < 65536 && tpw <= c.ntmax &&
        wgrad_lds(Ca, Cc, k, s, c.wt) <= 64 * 1024)
      return i;
  }
  return -1;
}

static int wgrad_chunks(int n, int Lp, int wt) { return n * ((Lp + wt - 1) / wt); }

// blocks (= partials) of stage 1: one resident round, one 8-wave block per CU
// (the staging registers and the accumulators take up to 256 VGPRs)
static int wgrad_blocks(int nchunk) { return std::max(1, std::min(nchunk, 256)); }

// an upper bound over every configuration (the smallest chunk has the most)
size_t wgrad_scratch_bytes(int n, int Lp, int nw) {
  const size_t G = (size_t)wgrad_blocks(wgrad_chunks(n, Lp, 64));
  const size_t ngroup = (G + WG - 1) / WG;
  size_t a = ((G * nw * sizeof(float)) + 255) & ~(size_t)255;
  return a + ngroup * nw * sizeof(double);
}

struct WgP {
  const float* P;
  const float* Q;
  int Ca, Lp, Cc, Lq, n, k, s, pad, tchunks, nchunk, qs;
  float* partial;  // [blocks][Ca*Cc*k]
};

typedef float wf32x4 __attribute__((ext_vector_type(4)));

// one chunk's K steps for a wave with NT accumulator tiles: K steps slice,
// slice + ksp, ... of 4 time steps each; every operand read is unconditional
// (rows and columns past the GEMM read zero rows)
template <int NT, int WT>
__device__ __forceinline__ void wgrad_mma(const float* Ps, const float* Qs, const int* aoff, const int* boff, int s,
                                          int slice, int ksp, int lk, wf32x4* acc) {
  const int nkk = WT / 4 / ksp;
  const float* pa = Ps + 4 * slice + lk;
  const float* qb = Qs + s * (4 * slice + lk);
  const int da = 4 * ksp, db = 4 * ksp * s;
#pragma unroll 4
  for (int it = 0; it < nkk; ++it) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
      acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[aoff[u]], qb[boff[u]], acc[u], 0, 0, 0);
    pa += da;
    qb += db;
  }
}

template <int WT, int PMAX, int QMAX, int NTMAX>
__global__ __launch_bounds__(WTH, 2) void wgrad_partial(WgP p) {
  extern __shared__ float lds[];
  constexpr int WPS = WT + 4;              // P row stride: rows 4 banks apart
  const int span = p.s * (WT - 1) + p.k;   // Q samples one chunk touches
  float* Ps = lds;                         // [Ca + 1][WPS], row Ca zero
  float* Qs = lds + (p.Ca + 1) * WPS;      // [Cc + 1][qs], row Cc zero
  const int tid = threadIdx.x;
  const int np = p.Ca * WT, nq = p.Cc * span;
  // this thread's Q elements (channel << 16 | position in the span), the
  // same for every chunk; -1 where the thread has none
  int qcu[QMAX];
#pragma unroll
  for (int i = 0; i < QMAX; ++i) {
    const int e = tid + WTH * i;
    const int c = e / span;
    qcu[i] = e < nq ? (c << 16) | (e - c * span) : -1;
  }
  // loads are unconditional, from addresses clamped into the tensors, so that
  // a chunk's loads are all in flight together; the staging store zeroes
  // what lies outside (rows past C, time past L, Q's zero padding)
  float pv[PMAX], qv[QMAX];
  auto fetch = [&](int chunk) {
    const int b = chunk / p.tchunks, t0 = (chunk - b * p.tchunks) * WT;
    const float* Pb = p.P + (int64_t)b * p.Ca * p.Lp;
    const float* Qb = p.Q + (int64_t)b * p.Cc * p.Lq;
#pragma unroll
    for (int i = 0; i < PMAX; ++i) {
      const int e = tid + WTH * i, a = min(e / WT, p.Ca - 1), t = min(t0 + e % WT, p.Lp - 1);
      pv[i] = Pb[(int64_t)a * p.Lp + t];
    }
    const int q0 = p.s * t0 - p.pad;
#pragma unroll
    for (int i = 0; i < QMAX; ++i) {
      const int c = qcu[i] >= 0 ? qcu[i] >> 16 : 0;
      const int q = min(max(q0 + (qcu[i] & 0xffff), 0), p.Lq - 1);
      qv[i] = Qb[(int64_t)c * p.Lq + q];
    }
  };
  // branch-free: a thread's slots past the chunk go to its own sink word, so
  // that every register of the batch is consumed on every path
  float* sink = Qs + (p.Cc + 1) * p.qs + tid;
  for (int e = tid; e < WPS; e += WTH) Ps[p.Ca * WPS + e] = 0.0f;
  for (int e = tid; e < p.qs; e += WTH) Qs[p.Cc * p.qs + e] = 0.0f;
  auto stage = [&](int chunk) {
    const int t0 = (chunk % p.tchunks) * WT, q0 = p.s * t0 - p.pad;
#pragma unroll
    for (int i = 0; i < PMAX; ++i) {
      const int e = tid + WTH * i;
      float* d = e < np ? Ps + (e / WT) * WPS + e % WT : sink;
      *d = t0 + e % WT < p.Lp ? pv[i] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < QMAX; ++i) {
      const int q = q0 + (qcu[i] & 0xffff);
      float* d = qcu[i] >= 0 ? Qs + (qcu[i] >> 16) * p.qs + (qcu[i] & 0xffff) : sink;
      *d = (q >= 0 && q < p.Lq) ? qv[i] : 0.0f;
    }
  };
  const int nk = p.Cc * p.k;               // GEMM columns
  const int MTa = (p.Ca + 15) / 16, NTn = (nk + 15) / 16, ntile = MTa * NTn;
  // wave groups splitting the K steps: as many as the idle waves allow
  const int ksp = wgrad_ksp(ntile);
  const int nwk = WNW / ksp;               // waves per group
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = wave / nwk, wl = wave - slice * nwk;
  const int lr = lane & 15, lk = lane >> 4;
  // this lane's LDS offsets for each of its tiles (tile u of the wave is
  // wl + nwk u): A row a = 16 mt + lr, B column n = 16 nt + lr = (c, j)
  int aoff[NTMAX], boff[NTMAX];
#pragma unroll
  for (int u = 0; u < NTMAX; ++u) {
    const int tile = wl + nwk * u;
    const int mt = tile / NTn, nt = tile - mt * NTn;
    const int a = 16 * mt + lr, nn = 16 * nt + lr;
    aoff[u] = (tile < ntile && a < p.Ca) ? a * WPS : p.Ca * WPS;
    boff[u] = (tile < ntile && nn < nk) ? (nn / p.k) * p.qs + (nn % p.k) : p.Cc * p.qs;
  }
  wf32x4 acc[NTMAX];
#pragma unroll
  for (int u = 0; u < NTMAX; ++u) acc[u] = wf32x4{0.f, 0.f, 0.f, 0.f};
  // this wave's tiles: wl, wl + nwk, ... below ntile
  const int mytiles = wl < ntile ? (ntile - wl + nwk - 1) / nwk : 0;
  const int G = gridDim.x;
  const int c0 = (int)((int64_t)p.nchunk * blockIdx.x / G), c1 = (int)((int64_t)p.nchunk * (blockIdx.x + 1) / G);
  if (c0 < c1) fetch(c0);
  for (int chunk = c0; chunk < c1; ++chunk) {
    __syncthreads();  // the previous chunk's reads are done
    stage(chunk);
    __syncthreads();
    if (chunk + 1 < c1) fetch(chunk + 1);  // in flight during this chunk's MFMAs
#define GW_WG_CASE(N)                                                          \
  case N:                                                                      \
    if constexpr (N <= NTMAX) wgrad_mma<N, WT>(Ps, Qs, aoff, boff, p.s, slice, ksp, lk, acc); \
    break;
    switch (mytiles) {  // wave-uniform
      GW_WG_CASE(1)
      GW_WG_CASE(2)
      GW_WG_CASE(3)
      GW_WG_CASE(4)
      GW_WG_CASE(5)
      GW_WG_CASE(6)
      GW_WG_CASE(7)
      default: break;
    }
#undef GW_WG_CASE
  }
  // groups 1.. hand their accumulators to group 0 through LDS, which adds
  // them in group order
  if (ksp > 1) {
    float* xs = lds;  // [group - 1][wl][u][lane][4]
    const int tpw = (ntile + nwk - 1) / nwk;
    __syncthreads();
    if (slice > 0)
#pragma unroll
      for (int u = 0; u < NTMAX; ++u) {
        if (u >= tpw) break;
        float* d = xs + ((((slice - 1) * nwk + wl) * tpw + u) * 64 + lane) * 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) d[r] = acc[u][r];
      }
    __syncthreads();
    if (slice == 0)
      for (int g = 1; g < ksp; ++g)
#pragma unroll
        for (int u = 0; u < NTMAX; ++u) {
          if (u >= tpw) break;
          const float* d = xs + ((((g - 1) * nwk + wl) * tpw + u) * 64 + lane) * 4;
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[u][r] += d[r];
        }
    if (slice > 0) return;
  }
  // D[row = 4 lk + r][col = lr] of tile u: weight (a, n)
  const int nw = p.Ca * nk;
  float* out = p.partial + (int64_t)blockIdx.x * nw;
#pragma unroll
  for (int u = 0; u < NTMAX; ++u) {
    const int tile = wl + nwk * u;
    if (tile >= ntile) break;
    const int mt = tile / NTn, nt = tile - mt * NTn;
    const int nn = 16 * nt + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int a = 16 * mt + 4 * lk + r;
      if (a < p.Ca && nn < nk) out[(int64_t)a * nk + nn] = acc[u][r];
    }
  }
}

// partials q of group g added in order q = 64 g, 64 g + 1, ...; the loads of
// 16 partials are issued together
__global__ __launch_bounds__(256) void wgrad_group(const float* partial, int nchunk, int nw,
                                                   double* mid) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int g = blockIdx.y;
  if (e >= nw) return;
  double acc = 0.0;
  const int q1 = min(nchunk, (g + 1) * WG);
  int q = g * WG;
  for (; q + 16 <= q1; q += 16) {
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = partial[(int64_t)(q + j) * nw + e];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc += (double)v[j];
  }
  for (; q < q1; ++q) acc += (double)partial[(int64_t)q * nw + e];
  mid[(int64_t)g * nw + e] = acc;
}

__global__ __launch_bounds__(256) void wgrad_final(const double* mid, int ngroup, int nw,
                                                   float* dw) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= nw) return;
  double acc = 0.0;
  int g = 0;
  for (; g + 8 <= ngroup; g += 8) {
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = mid[(int64_t)(g + j) * nw + e];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc += v[j];
  }
  for (; g < ngroup; ++g) acc += mid[(int64_t)g * nw + e];
  dw[e] = (float)acc;
}

hipError_t launch_wgrad(const float* P, int Ca, int Lp, const float* Q, int Cc, int Lq, int n,
                        int k, int stride, int pad, void* scratch, float* dw, hipStream_t st) {
  const int cfg = wgrad_cfg(Ca, Cc, k, stride);
  const int nw = Ca * Cc * k;
  // every accumulator tile of the GEMM must have a register slot in its wave
  if (cfg < 0 || ((Ca + 15) / 16) * ((Cc * k + 15) / 16) > WNW * WTPW) return hipErrorInvalidValue;
  const int wt = kWgCfg[cfg].wt;
  WgP p;
  p.P = P;
  p.Q = Q;
  p.Ca = Ca;
  p.Lp = Lp;
  p.Cc = Cc;
  p.Lq = Lq;
  p.n = n;
  p.k = k;
  p.s = stride;
  p.pad = pad;
  p.tchunks = (Lp + wt - 1) / wt;
  p.nchunk = wgrad_chunks(n, Lp, wt);
  p.qs = wgrad_qs(stride * (wt - 1) + k);
  const int G = wgrad_blocks(p.nchunk);
  const int ngroup = (G + WG - 1) / WG;
  p.partial = reinterpret_cast<float*>(scratch);
  double* mid = reinterpret_cast<double*>(reinterpret_cast<char*>(scratch) +
                                          ((((size_t)G * nw * sizeof(float)) + 255) & ~(size_t)255));
  const size_t lds = wgrad_lds(Ca, Cc, k, stride, wt);
  switch (cfg) {
    case 0: hipLaunchKernelGGL((wgrad_partial<1024, 8, 24, 3>), dim3(G), dim3(WTH), lds, st, p); break;
    case 1: hipLaunchKernelGGL((wgrad_partial<512, 8, 24, 3>), dim3(G), dim3(WTH), lds, st, p); break;
    case 2: hipLaunchKernelGGL((wgrad_partial<256, 8, 24, 3>), dim3(G), dim3(WTH), lds, st, p); break;
    case 3: hipLaunchKernelGGL((wgrad_partial<128, 8, 12, 3>), dim3(G), dim3(WTH), lds, st, p); break;
    case 4: hipLaunchKernelGGL((wgrad_partial<64, 8, 12, 7>), dim3(G), dim3(WTH), lds, st, p); break;
    default: hipLaunchKernelGGL((wgrad_partial<64, 16, 24, 7>), dim3(G), dim3(WTH), lds, st, p); break;
  }
  hipLaunchKernelGGL(wgrad_group, dim3((nw + 255) / 256, ngroup), dim3(256), 0, st, p.partial,
                     G, nw, mid);
  hipLaunchKernelGGL(wgrad_final, dim3((nw + 255) / 256), dim3(256), 0, st, mid, ngroup, nw, dw);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Band-passed MSE.  With r = strain - noise and the DFT basis
// cos/sin(2 pi k t / W) of the band bins k_lo..k_hi,
//   ||P r||^2 = sum_k c_k (A_k^2 + B_k^2),  A_k = <r, cos_k>, B_k = <r, sin_k>,
//   P r[t]    = sum_k c_k (A_k cos_k[t] + B_k sin_k[t]),
// with c_k = 2/W (c_k = 1/W for k = 0 or k = W/2).  Angles are reduced
// exactly in integers, m = (k t mod W), before the sin/cos evaluation; the
// index advances by a constant per step (one compare and subtract).
//
// Both directions are matrix products with the basis, which is evaluated in
// registers where the matrix cores want it: a lane's (cos, sin) pair is its
// element of two operands, and serves 16 windows a matrix instruction.
//
// Measured, 32 windows of 32768, 81 bins, loss and gradient: one thread per
// (sample, bin) with vector FP64 sums, four windows a basis value 99 us;
// these kernels 44 us.  Left: the basis evaluations, the FP64 products at
// half of the vector FP32 rate (5 us), and three dependent launches.  Calls of up
// to four windows leave the matrix instructions, whose rows they do not fill, to
// FP64 products in vector registers (the rules are at the end).
// ---------------------------------------------------------------------------
namespace bp {

typedef double f64x4 __attribute__((ext_vector_type(4)));
// k t mod W
__device__ __forceinline__ int mulmod(int k, int t, int W) {
  if (W < 1 << 24) {  // the product is exact, the quotient off by one at most
    const double v = (double)k * (double)t;
    const double r = fma(-floor(v * (1.0 / (double)W)), (double)W, v);
    int m = (int)r;
    if (m < 0) m += W;
    return m >= W ? m - W : m;
  }
  return (int)((int64_t)k * t % W);
}

}  // namespace bp

// Projections: D[window][bin] += r[window][t] basis[t][bin] over a slice of the
// samples, on v_mfma_f64_16x16x4_f64: FP32 residuals and basis values, exact
// products, FP64 sums.  A block takes 16 bins (cos and sin) of 16 MT windows;
// its eight waves take 16 samples each of every 128 of the slice, lane l
// sample 4 (l / 16) + e in step e.  The waves' sums are added through LDS.
template <int MT>
__global__ __launch_bounds__(512) void bp_project(const float* strain, const float* noise, int n, int nb, int W,
                                                  int k_lo, int S, double* partial, float* proj) {
  using namespace bp;
  __shared__ double red[4][MT * 2 * 4 * 64];
  const int tile = blockIdx.x / S, slice = blockIdx.x - tile * S;
  const int b0 = blockIdx.y * 16 * MT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int rounds = (W + 127) / 128;
  const int c0 = (int)((int64_t)rounds * slice / S), c1 = (int)((int64_t)rounds * (slice + 1) / S);
  const bool vec = ((W & 3) | ((reinterpret_cast<uintptr_t>(strain) | reinterpret_cast<uintptr_t>(noise)) & 15)) == 0;
  const int k = k_lo + min(16 * tile + lr, nb - 1);
  int t = 128 * c0 + 16 * wave + 4 * lk;
  int m = mulmod(k, t, W);
  const int step = mulmod(k, 128, W);
  f64x4 acc[MT][2];
#pragma unroll
  for (int g = 0; g < MT; ++g) acc[g][0] = acc[g][1] = f64x4{0.0, 0.0, 0.0, 0.0};
  const float* sp[MT];
  const float* np[MT];
#pragma unroll
  for (int g = 0; g < MT; ++g) {  // rows past n read the last one; their sums are dropped
    const int64_t o = (int64_t)min(b0 + 16 * g + lr, n - 1) * W;
    sp[g] = strain + o;
    np[g] = noise + o;
  }
  float r[MT][4], nx[MT][4];
  auto load = [&](float (&v)[MT][4], int t) {
#pragma unroll
    for (int g = 0; g < MT; ++g) {
      if (vec && t + 4 <= W) {
        const float4 a = *reinterpret_cast<const float4*>(sp[g] + t), b = *reinterpret_cast<const float4*>(np[g] + t);
        v[g][0] = a.x - b.x;
        v[g][1] = a.y - b.y;
        v[g][2] = a.z - b.z;
        v[g][3] = a.w - b.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[g][e] = t + e < W ? sp[g][t + e] - np[g][t + e] : 0.0f;
      }
    }
  };
  const float twoW = 2.0f / (float)W;
  if (c0 < c1) load(nx, t);
  for (int c = c0; c < c1; ++c, t += 128) {
#pragma unroll
    for (int g = 0; g < MT; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) r[g][e] = nx[g][e];
    if (c + 1 < c1) load(nx, t + 128);
    int me = m;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float sn, cs;
      sincospif(twoW * (float)me, &sn, &cs);
#pragma unroll
      for (int g = 0; g < MT; ++g) {
        acc[g][0] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)r[g][e], (double)cs, acc[g][0], 0, 0, 0);
        acc[g][1] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)r[g][e], (double)sn, acc[g][1], 0, 0, 0);
      }
      me += k;
      if (me >= W) me -= W;
    }
    m += step;
    if (m >= W) m -= W;
  }
  // waves 4 .. 7 hand over to 0 .. 3, whose sums are added in wave order
  auto slot = [&](int g, int q, int i) { return ((g * 2 + q) * 4 + i) * 64 + lane; };
  if (wave >= 4)
#pragma unroll
    for (int g = 0; g < MT; ++g)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wave - 4][slot(g, q, i)] = acc[g][q][i];
  __syncthreads();
  if (wave < 4)
#pragma unroll
    for (int g = 0; g < MT; ++g)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wave][slot(g, q, i)] += acc[g][q][i];
  __syncthreads();
  // lane 16 lk + bin holds windows 4 i + lk in element i
  for (int e = tid; e < MT * 512; e += 512) {
    const int q = e & 1, bb = (e >> 1) % (16 * MT), bin = e / (32 * MT);
    const int o = (((bb >> 4) * 2 + q) * 4 + ((bb & 15) >> 2)) * 64 + 16 * (bb & 3) + bin;
    const int kk = 16 * tile + bin, b = b0 + bb;
    if (kk < nb && b < n) {
      const double v = ((red[0][o] + red[1][o]) + red[2][o]) + red[3][o];
      const int64_t at = ((int64_t)kk * n + b) * 2 + q;
      if (S == 1)
        proj[at] = (float)v;
      else
        partial[slice * (2 * (int64_t)n * nb) + at] = v;
    }
  }
}

// The same for NW windows, up to four: there the matrix instruction's 16 rows
// are mostly empty, and two of it cost as much as the basis values.  A wave
// takes one bin over a slice of the samples, its lanes every 64th, with FP64
// products and sums in vector registers; the lanes' sums are added in a fixed tree.
template <int NW>
__global__ __launch_bounds__(256) void bp_project_few(const float* strain, const float* noise, int nb, int W, int k_lo,
                                                      int S, double* partial, float* proj) {
  using namespace bp;
  const int tile = (int)blockIdx.x / S, slice = (int)blockIdx.x - tile * S;
  const int lane = threadIdx.x & 63;
  const int kk = 4 * tile + (int)(threadIdx.x >> 6), k = k_lo + kk;
  if (kk >= nb) return;  // wave-uniform; the kernel has no barrier
  const int rounds = (W + 63) / 64;
  const int c0 = (int)((int64_t)rounds * slice / S), c1 = (int)((int64_t)rounds * (slice + 1) / S);
  const int step = mulmod(k, 64, W), t1 = min(64 * c1, W);
  int m = mulmod(k, min(64 * c0 + lane, W - 1), W);
  double a[NW], b[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) a[w] = b[w] = 0.0;
  const float twoW = 2.0f / (float)W;
#pragma unroll 2
  for (int t = 64 * c0 + lane; t < t1; t += 64) {
    float sn, cs;
    sincospif(twoW * (float)m, &sn, &cs);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const double r = (double)(strain[(int64_t)w * W + t] - noise[(int64_t)w * W + t]);
      a[w] = fma(r, (double)cs, a[w]);
      b[w] = fma(r, (double)sn, b[w]);
    }
    m += step;
    if (m >= W) m -= W;
  }
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    for (int off = 32; off > 0; off >>= 1) {
      a[w] += __shfl_down(a[w], off, 64);
      b[w] += __shfl_down(b[w], off, 64);
    }
    const int64_t at = (int64_t)kk * NW + w;
    if (lane != 0) continue;
    if (S == 1)
      reinterpret_cast<float2*>(proj)[at] = make_float2((float)a[w], (float)b[w]);
    else
      reinterpret_cast<double2*>(partial)[slice * (int64_t)nb * NW + at] = make_double2(a[w], b[w]);
  }
}

// proj[bin][window][2] = the slices' sums, rounded once: a block takes 64
// values, its four waves a quarter of the slices each, in order
__global__ __launch_bounds__(256) void bp_final(const double* partial, int64_t nv, int S, float* proj) {
  __shared__ double s[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  const int s1 = S * (wave + 1) / 4;
  double acc = 0.0;
  if (e < nv) {
    int g = S * wave / 4;
    for (; g + 8 <= s1; g += 8) {
      double v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = partial[(int64_t)(g + j) * nv + e];
#pragma unroll
      for (int j = 0; j < 8; ++j) acc += v[j];
    }
    for (; g < s1; ++g) acc += partial[(int64_t)g * nv + e];
  }
  s[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && e < nv) proj[e] = (float)(((s[0][lane] + s[1][lane]) + s[2][lane]) + s[3][lane]);
}

// weight of bin k against the others': c_k W / 2, exact
__device__ __forceinline__ float bin_weight(int k, int W) { return k == 0 || 2 * k == W ? 0.5f : 1.0f; }

// in a block of 256 threads, or by the first 256 of a larger one
__device__ __forceinline__ void bp_loss_block(const float* proj, int n, int nb, int W, int k_lo, float* loss) {
  __shared__ double sv[256];
  const int tid = threadIdx.x;
  double s = 0.0;
  const int64_t np = (int64_t)n * nb;
  const double first = bin_weight(k_lo, W), last = bin_weight(k_lo + nb - 1, W);
  if (tid < 256) {
#pragma unroll 4
    for (int64_t e = tid; e < np; e += 256) {
      const float2 v = reinterpret_cast<const float2*>(proj)[e];
      s += (e < n ? first : e >= np - n ? last : 1.0) * ((double)v.x * v.x + (double)v.y * v.y);
    }
    sv[tid] = s;
  }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) sv[tid] += sv[tid + w];
    __syncthreads();
  }
  if (tid == 0) loss[0] = (float)(sv[0] * (2.0 / (double)W) / ((double)n * W));
}

__global__ __launch_bounds__(256) void bp_loss(const float* proj, int n, int nb, int W, int k_lo, float* loss) {
  bp_loss_block(proj, n, nb, W, k_lo, loss);
}

// bp_final and bp_loss in one block, bit for bit, for up to eight slices: the loss
// alone of a small call, where a launch more is a tenth of its time.
__global__ __launch_bounds__(1024) void bp_final_loss(const double* partial, int nv, int S, float* proj, int n, int nb,
                                                      int W, int k_lo, float* loss) {
#pragma unroll 2
  for (int e = threadIdx.x; e < nv; e += 1024) {
    double v[8], q[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int g = 0; g < 8; ++g) v[g] = g < S ? partial[(int64_t)g * nv + e] : 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int g = 0; g < 8; ++g)
        if (g >= S * w / 4 && g < S * (w + 1) / 4) q[w] += v[g];
    proj[e] = (float)(((q[0] + q[1]) + q[2]) + q[3]);
  }
  __syncthreads();
  bp_loss_block(proj, n, nb, W, k_lo, loss);
}

// dL/dnoise[window][t] = scale * sum over bins of weight (A cos[t] + B sin[t]),
// on the same instruction: a wave takes 16 samples of 16 MT windows and four
// bins a step.  (With FP32 sums it took 11 us instead of 17, and had up to 1.4 times
// the error of the kernel before it.)  SPLIT: the block's four waves take a
// quarter of the bins each of the same 16 samples, for launches of few blocks; else
// 16 samples each.  The last block of the first row computes the loss, if that is
// asked for.
template <int MT, bool SPLIT>
__global__ __launch_bounds__(256) void bp_grad(const float* proj, int n, int nb, int W, int k_lo, double scale,
                                               float* dnoise, float* loss) {
  using namespace bp;
  if (loss && blockIdx.x == gridDim.x - 1) {
    if (blockIdx.y == 0) bp_loss_block(proj, n, nb, W, k_lo, loss);
    return;
  }
  __shared__ double red[SPLIT ? 4 : 1][SPLIT ? MT * 4 * 64 : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int b0 = blockIdx.y * 16 * MT;
  const int t = SPLIT ? blockIdx.x * 16 + lr : blockIdx.x * 64 + 16 * wave + lr, tc = min(t, W - 1);
  const int steps = (nb + 7) / 8;  // of eight bins
  const int k0 = SPLIT ? 8 * (steps * wave / 4) : 0, k1 = SPLIT ? min(8 * (steps * (wave + 1) / 4), nb) : nb;
  int m = mulmod(min(k_lo + k0 + lk, W - 1), tc, W);
  const int step = mulmod(4, tc, W);
  const float twoW = 2.0f / (float)W;
  const float2* src[MT];
#pragma unroll
  for (int g = 0; g < MT; ++g)
    src[g] = reinterpret_cast<const float2*>(proj) + min(b0 + 16 * g + lr, n - 1);
  f64x4 acc[MT][2];
#pragma unroll
  for (int g = 0; g < MT; ++g)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[g][q] = f64x4{0.0, 0.0, 0.0, 0.0};
  float2 next[2][MT];
  auto load = [&](int kk0) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int g = 0; g < MT; ++g) next[h][g] = src[g][(int64_t)min(kk0 + 4 * h + lk, nb - 1) * n];
  };
  load(k0);
  for (int kk0 = k0; kk0 < k1; kk0 += 8) {
    float2 v[2][MT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int g = 0; g < MT; ++g) v[h][g] = next[h][g];
    load(kk0 + 8);  // in flight during this step's basis values
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kk = kk0 + 4 * h + lk;
      const float w = bin_weight(k_lo + kk, W);
      float sn, cs;
      sincospif(twoW * (float)m, &sn, &cs);
#pragma unroll
      for (int g = 0; g < MT; ++g) {
        // bins past the band have zero coefficients, whatever was read
        v[h][g] = kk < nb ? make_float2(w * v[h][g].x, w * v[h][g].y) : make_float2(0.f, 0.f);
        acc[g][0] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[h][g].x, (double)cs, acc[g][0], 0, 0, 0);
        acc[g][1] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[h][g].y, (double)sn, acc[g][1], 0, 0, 0);
      }
      m += step;
      if (m >= W) m -= W;
    }
  }
  if constexpr (SPLIT) {
#pragma unroll
    for (int g = 0; g < MT; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[wave][(4 * g + i) * 64 + lane] = acc[g][0][i] + acc[g][1][i];
    __syncthreads();
    for (int e = threadIdx.x; e < MT * 256; e += 256) {
      const int l = e & 63, b = b0 + 4 * (e >> 6) + (l >> 4), u = blockIdx.x * 16 + (l & 15);
      if (b < n && u < W)
        dnoise[(int64_t)b * W + u] = (float)(scale * (((red[0][e] + red[1][e]) + red[2][e]) + red[3][e]));
    }
  } else {
    if (t >= W) return;
#pragma unroll
    for (int g = 0; g < MT; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int b = b0 + 16 * g + 4 * i + lk;
        if (b < n) dnoise[(int64_t)b * W + t] = (float)(scale * (acc[g][0][i] + acc[g][1][i]));
      }
  }
}

// The same for NW windows, up to four, as bp_project_few is: a block takes 64
// samples, its eight waves an eighth of the bins each, whose sums are added in
// wave order.
template <int NW>
__global__ __launch_bounds__(512) void bp_grad_few(const float* __restrict__ proj, int nb, int W, int k_lo, double scale,
                                                   float* __restrict__ dnoise, float* loss) {
  using namespace bp;
  if (loss && blockIdx.x == gridDim.x - 1) {
    bp_loss_block(proj, NW, nb, W, k_lo, loss);
    return;
  }
  __shared__ double red[8][NW * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.x * 64 + lane, tc = min(t, W - 1);
  const int k0 = (int)((int64_t)nb * wave / 8), k1 = (int)((int64_t)nb * (wave + 1) / 8);
  int m = mulmod(min(k_lo + k0, W - 1), tc, W);
  const float twoW = 2.0f / (float)W;
  double acc[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) acc[w] = 0.0;
#pragma unroll 2
  for (int kk = k0; kk < k1; ++kk) {
    const float bw = bin_weight(k_lo + kk, W);
    float sn, cs;
    sincospif(twoW * (float)m, &sn, &cs);
    const float2* v = reinterpret_cast<const float2*>(proj) + (int64_t)kk * NW;  // wave-uniform
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      acc[w] = fma((double)(bw * v[w].x), (double)cs, acc[w]);
      acc[w] = fma((double)(bw * v[w].y), (double)sn, acc[w]);
    }
    m += tc;
    if (m >= W) m -= W;
  }
#pragma unroll
  for (int w = 0; w < NW; ++w) red[wave][w * 64 + lane] = acc[w];
  __syncthreads();
  for (int e = threadIdx.x; e < NW * 64; e += 512) {
    double a = red[0][e];
#pragma unroll
    for (int w = 1; w < 8; ++w) a += red[w][e];
    const int u = blockIdx.x * 64 + (e & 63);
    if (u < W) dnoise[(int64_t)(e >> 6) * W + u] = (float)(scale * a);
  }
}

namespace bp {
// Windows per block: 32, or 16 where that covers them all.
int windows(int n) { return n > 16 ? 32 : 16; }
// Up to four windows take the kernels without matrix instructions.  Measured (us
// of the device, loss and gradient; loss alone): one window of 32768, 20 .. 500 Hz at
// 4096 samples a second (3841 bins) 271 and 144 (matrix 617 and 271), 55 .. 65 Hz (81
// bins) 18 and 18 (27 and 19); four windows of 32768, 3841 bins: 417 and 234 (616 and
// 275); five windows, every bin, in them 2426 and 1237: a second batch of four would
// take 1600 more.
bool few(int n) { return n <= 4; }
// The gradient so only for launches of 128 blocks or more: four windows of 4096,
// every bin, 100 us against 64 for bp_grad with its bins split; one of 8192, 134
// against 224.
bool few_grad(int n, int W) { return few(n) && W >= 8192; }
// bp_grad splits its bins where that fills the chip: 32 windows of 8192, 961 bins
// (128 blocks unsplit) 127 -> 74 us, of 16384 (256) 290 -> 236, 32 of 512, 257 bins,
// 37 -> 20, one of 2048, 241 bins, 25 -> 14, 16 of 8192, 81 bins, 19 -> 16.  Few bins
// are not worth their sums' exchange: 81 in 512 blocks 41.9 against 42.8.
bool split(int n, int W, int nb) {
  const int64_t blocks = (int64_t)((W + 63) / 64) * ((n + windows(n) - 1) / windows(n));
  return blocks < 1024 && nb >= (blocks <= 256 ? 64 : 256);
}
// Slices of the samples.  bp_project: as many as make 512 blocks (16 waves a CU),
// of 128 samples at least, in multiples of eight so that a slice's bin tiles,
// which read the same samples, meet in one XCD's cache.  bp_project_few: as many
// as make 4096 waves, of 512 samples at least, and up to 2048 samples one, which
// needs no launch to add them (one of 1024, 257 bins, loss and gradient: 18.7 ->
// 16.6 us; one of 2048, 1025 bins, the loss alone: 13.2 -> 11.9).
int slices(int n, int W, int nb) {
  if (few(n) && W <= 2048) return 1;
  if (few(n)) return (int)std::max<int64_t>(1, std::min<int64_t>(4096 / nb, (W + 63) / 64 / 8));
  const int64_t blocks = (int64_t)((nb + 15) / 16) * ((n + windows(n) - 1) / windows(n));
  const int64_t s = std::max<int64_t>(1, std::min<int64_t>(512 / blocks, (W + 127) / 128));
  return (int)(s >= 8 ? s / 8 * 8 : s);
}
// Whether the loss alone takes bp_final_loss: 16 windows of 1024, 121 bins (3872
// values of eight slices) 15.7 us of the device against 13.0 in three launches, but
// 17.3 a call against 19 on the host; twice the windows 21.7 against 15.6, and 20.6
// a call against 18.9.
bool one_block(int64_t nv, int S) { return S > 1 && S <= 8 && nv <= 4096; }
}  // namespace bp

// The projections, and before them the slices' FP64 sums if there is more than
// one slice (then at most 4 MiB).
size_t bandpass_ws_bytes(int n, int W, int nb) {
  const int S = bp::slices(n, W, nb);
  return 8 * (size_t)n * nb * (S > 1 ? 1 + 2 * (size_t)S : 1);
}

template <int NW>
static void launch_few(bool grad, int nb, int W, int k_lo, int S, const float* strain, const float* noise, double* partial,
                       float* proj, double scale, float* dnoise, float* loss, hipStream_t st) {
  if (!grad)
    hipLaunchKernelGGL(bp_project_few<NW>, dim3((nb + 3) / 4 * S), dim3(256), 0, st, strain, noise, nb, W, k_lo, S,
                       partial, proj);
  else
    hipLaunchKernelGGL(bp_grad_few<NW>, dim3((W + 63) / 64 + (loss ? 1 : 0)), dim3(512), 0, st, proj, nb, W, k_lo, scale,
                       dnoise, loss);
}

hipError_t launch_bandpass(int n, int W, int k_lo, int k_hi, const float* strain,
                           const float* noise, void* ws, float* loss, float* dnoise,
                           hipStream_t st) {
  const int nb = k_hi - k_lo + 1;
  if (nb <= 0) return hipErrorInvalidValue;
  const int nw = bp::windows(n), S = bp::slices(n, W, nb), gy = (n + nw - 1) / nw;
  const int64_t nv = 2 * (int64_t)n * nb;
  const double scale = -2.0 / ((double)n * W) * (2.0 / (double)W);
  double* partial = reinterpret_cast<double*>(ws);
  float* proj = S > 1 ? reinterpret_cast<float*>(partial + S * nv) : reinterpret_cast<float*>(ws);
  const auto few = [&](bool grad) {
    const auto f = n == 1 ? launch_few<1> : n == 2 ? launch_few<2> : n == 3 ? launch_few<3> : launch_few<4>;
    f(grad, nb, W, k_lo, S, strain, noise, partial, proj, scale, dnoise, loss, st);
  };
  const dim3 pg((nb + 15) / 16 * S, gy);  // 16-bin tiles x slices, windows
  if (bp::few(n))
    few(false);
  else if (nw == 32)
    hipLaunchKernelGGL(bp_project<2>, pg, dim3(512), 0, st, strain, noise, n, nb, W, k_lo, S, partial, proj);
  else
    hipLaunchKernelGGL(bp_project<1>, pg, dim3(512), 0, st, strain, noise, n, nb, W, k_lo, S, partial, proj);
  if (!dnoise && loss && bp::one_block(nv, S)) {
    hipLaunchKernelGGL(bp_final_loss, dim3(1), dim3(1024), 0, st, partial, (int)nv, S, proj, n, nb, W, k_lo,
                       loss);
    return hipGetLastError();
  }
  if (S > 1) hipLaunchKernelGGL(bp_final, dim3((unsigned)((nv + 63) / 64)), dim3(256), 0, st, partial, nv, S, proj);
  if (!dnoise) {
    if (loss) hipLaunchKernelGGL(bp_loss, dim3(1), dim3(256), 0, st, proj, n, nb, W, k_lo, loss);
  } else if (bp::few_grad(n, W)) {
    few(true);
  } else {
    const bool split = bp::split(n, W, nb);
    const dim3 gg((split ? (W + 15) / 16 : (W + 63) / 64) + (loss ? 1 : 0), gy);
    const auto grad = nw == 32 ? (split ? bp_grad<2, true> : bp_grad<2, false>) : split ? bp_grad<1, true> : bp_grad<1, false>;
    hipLaunchKernelGGL(grad, gg, dim3(256), 0, st, proj, n, nb, W, k_lo, scale, dnoise, loss);
  }
  return hipGetLastError();
}

}  // namespace gw
