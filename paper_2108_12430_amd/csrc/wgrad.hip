// Weight gradients of the reference DeepClean network's layers, with the
// batch-normalisation transforms applied as the operands are staged.
//
//   dw[a][c][j] = sum over windows and t of P[a][t] Q[c][s t - 3 + j]
//
// (P = dL/dz and Q = layer input for a conv; P = layer input and Q = dL/dz for
// a transposed conv), a split-K GEMM D[a][n = 7 c + j] over K = (window, time)
// on v_mfma_f32_16x16x4_f32 (exact FP32 products, FP32 accumulation).  The
// layer input is tanh(BN(z)) and dL/dz comes from dh = g (1 - a^2) and z, so
// neither is ever written to memory.
//
// Layout: P rows [channel][time] in LDS, Q rows the same, for stride 2 split
// by parity, so that a tap's samples of consecutive t are consecutive.  A K
// step takes 16 times: lane l holds t = 16 ks + 4 (l / 16) + e in element e,
// one 16-byte read of P and two paired 4-byte reads of Q (a tap shifts Q by
// 0..3 samples, so its reads are not 16-byte aligned) for four MFMAs.  The
// first version read one 4-byte operand per MFMA and operand and was bound by
// LDS issue.  Waves take K slices of a chunk (and shares of the columns where
// the accumulators would not fit), so a P fragment serves all of a wave's
// columns.  Each thread holds the next chunk's loads while the MFMAs run.
// Block sums are written as FP32 partials; one launch adds the partials of
// every layer in FP64 in a fixed order.
//
// Measured, batch 32 x 21 x 32768, all nine layers with their reductions: 384
// us with operands read from memory as they are and a launch pair per layer
// for the reduction, 302 us here, without the 190 us that wrote dz and the
// activations.
#include "internal.h"

namespace gw {
namespace wg2 {

typedef float f32x4 __attribute__((ext_vector_type(4)));

enum Mode : int { RAW = 0, ACT = 1, DZ = 2 };

template <int CA_, int CC_, int S_, int WT_, int NW_, int PM_, int QM_>
struct Cfg {
  static constexpr int CA = CA_, CC = CC_, S = S_, WT = WT_, NW = NW_, PM = PM_, QM = QM_;
  static constexpr int NTHR = 64 * NW;
  static constexpr int NK = CC * 7, MA = (CA + 15) / 16, NB = (NK + 15) / 16;
  static constexpr int KC = WT / 16;                    // K steps per chunk
  static constexpr int NS = KC < NW ? KC : NW;          // K slices
  static constexpr int NGR = NW / NS;                   // column groups
  static constexpr int NBW = (NB + NGR - 1) / NGR;      // column tiles per wave
  static constexpr int PS = WT + 4;                     // P row stride (floats): an odd multiple of 16 bytes
  static constexpr int QW = S * WT + 8;                 // Q samples per channel and chunk
  static constexpr int QP = S == 2 ? QW / 2 + 4 : QW + 4;  // Q row stride
  static constexpr int QROWS = S * CC;
  static constexpr int STAGE = CA * PS + QROWS * QP;
  static constexpr int RED = (NS / 2) * NGR * MA * NBW * 256;
  static constexpr int LDS = STAGE > RED ? STAGE : RED;
  static constexpr int IP = (CA * WT / 4 + NTHR - 1) / NTHR;
  static constexpr int IQ = (CC * QW / 4 + NTHR - 1) / NTHR;
  static_assert(WT % 16 == 0 && KC % NS == 0 && NW % NS == 0 && (NS & (NS - 1)) == 0, "slices");
};

struct Opnd {
  const float* x;
  BnBwdP bn;
};

struct P2 {
  Opnd p, q;
  int n, Lp, Lq, tchunks, nchunk;
  float* partial;  // [blocks][CA * NK]
};

// constants of a transformed operand, [6][C]
template <int C, int M>
__device__ __forceinline__ void consts(float* cb, const BnBwdP& q, int tid) {
  if (M == RAW || tid >= C) return;
  const float is = q.bn.invstd[tid], g = q.bn.gamma[tid];
  cb[tid] = q.bn.mean[tid];
  cb[C + tid] = is;
  cb[2 * C + tid] = g;
  cb[3 * C + tid] = M == DZ ? g * is : q.bn.beta[tid];
  if (M == DZ) {
    cb[4 * C + tid] = q.sum_dh[tid] * q.invN;
    cb[5 * C + tid] = q.sum_dhx[tid] * q.invN;
  }
}

// four samples [t, t + 4) of row `row` (zeros outside [0, L))
__device__ __forceinline__ float4 load4(const float* x, int64_t row, int L, int t, bool vec) {
  const float* r = x + row * L;
  if (vec && t >= 0 && t + 4 <= L) return *reinterpret_cast<const float4*>(r + t);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (t >= 0 && t < L) v.x = r[t];
  if (t + 1 >= 0 && t + 1 < L) v.y = r[t + 1];
  if (t + 2 >= 0 && t + 2 < L) v.z = r[t + 2];
  if (t + 3 >= 0 && t + 3 < L) v.w = r[t + 3];
  return v;
}

template <int C, int M>
__device__ __forceinline__ float4 transform(float4 v, const float4& z, const float* cb, int c, int t, int L) {
  if (M == RAW) return v;
  const float m = cb[c], is = cb[C + c], g = cb[2 * C + c], be = cb[3 * C + c];
  float* d = &v.x;
  const float* dz = &z.x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float y = M == ACT ? bn_tanh_one(d[j], m, is, g, be)
                             : bn_dz_one(d[j], dz[j], m, is, be, cb[4 * C + c], cb[5 * C + c]);
    d[j] = t + j >= 0 && t + j < L ? y : 0.0f;
  }
  return v;
}

}  // namespace wg2

template <class K>
__global__ __launch_bounds__(K::NTHR, 4) void wgrad2(wg2::P2 p) {
  using namespace wg2;
  __shared__ __attribute__((aligned(16))) float lds[K::LDS];
  __shared__ float cp[K::PM == RAW ? 1 : 6 * K::CA], cq[K::QM == RAW ? 1 : 6 * K::CC];
  float* Ps = lds;
  float* Qs = lds + K::CA * K::PS;
  const int tid = threadIdx.x;
  const bool vp = ((p.Lp & 3) | (reinterpret_cast<uintptr_t>(p.p.x) & 15) |
                   (K::PM == DZ ? reinterpret_cast<uintptr_t>(p.p.bn.z) & 15 : 0)) == 0;
  const bool vq = ((p.Lq & 3) | (reinterpret_cast<uintptr_t>(p.q.x) & 15) |
                   (K::QM == DZ ? reinterpret_cast<uintptr_t>(p.q.bn.z) & 15 : 0)) == 0;
  consts<K::CA, K::PM>(cp, p.p.bn, tid);
  consts<K::CC, K::QM>(cq, p.q.bn, tid);
  float4 pv[K::IP], pz[K::PM == DZ ? K::IP : 1], qv[K::IQ], qz[K::QM == DZ ? K::IQ : 1];
  constexpr int PC = K::WT / 4, QC = K::QW / 4;  // float4 items per row
  auto fetch = [&](int chunk) {
    const int b = chunk / p.tchunks, t0 = (chunk - b * p.tchunks) * K::WT;
#pragma unroll
    for (int i = 0; i < K::IP; ++i) {
      const int e = tid + K::NTHR * i, a = e / PC, t = t0 + 4 * (e - a * PC);
      if (e < K::CA * PC) {
        pv[i] = load4(p.p.x, (int64_t)b * K::CA + a, p.Lp, t, vp);
        if (K::PM == DZ) pz[i] = load4(p.p.bn.z, (int64_t)b * K::CA + a, p.Lp, t, vp);
      }
    }
#pragma unroll
    for (int i = 0; i < K::IQ; ++i) {
      const int e = tid + K::NTHR * i, c = e / QC, q = K::S * t0 - 4 + 4 * (e - c * QC);
      if (e < K::CC * QC) {
        qv[i] = load4(p.q.x, (int64_t)b * K::CC + c, p.Lq, q, vq);
        if (K::QM == DZ) qz[i] = load4(p.q.bn.z, (int64_t)b * K::CC + c, p.Lq, q, vq);
      }
    }
  };
  auto stage = [&](int chunk) {
    const int t0 = chunk % p.tchunks * K::WT;
#pragma unroll
    for (int i = 0; i < K::IP; ++i) {
      const int e = tid + K::NTHR * i, a = e / PC, r = 4 * (e - a * PC);
      if (e < K::CA * PC)
        *reinterpret_cast<float4*>(Ps + a * K::PS + r) =
            transform<K::CA, K::PM>(pv[i], pz[K::PM == DZ ? i : 0], cp, a, t0 + r, p.Lp);
    }
#pragma unroll
    for (int i = 0; i < K::IQ; ++i) {
      const int e = tid + K::NTHR * i, c = e / QC, r = 4 * (e - c * QC);
      if (e < K::CC * QC) {
        const float4 v =
            transform<K::CC, K::QM>(qv[i], qz[K::QM == DZ ? i : 0], cq, c, K::S * t0 - 4 + r, p.Lq);
        if (K::S == 2) {
          *reinterpret_cast<float2*>(Qs + 2 * c * K::QP + r / 2) = make_float2(v.x, v.z);
          *reinterpret_cast<float2*>(Qs + (2 * c + 1) * K::QP + r / 2) = make_float2(v.y, v.w);
        } else {
          *reinterpret_cast<float4*>(Qs + c * K::QP + r) = v;
        }
      }
    }
  };
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int slice = wave / K::NGR, grp = wave - slice * K::NGR;
  // rows and columns past the GEMM read the last real one; their sums are dropped
  static_assert(K::MA == 1 || K::CA % 16 == 0, "whole row tiles");
  const float* ap = Ps + (lr < K::CA ? lr : K::CA - 1) * K::PS + 4 * lk;
  // sample of (t, tap j): S t - 3 + j, staged from S t0 - 4 on
  const float* bp[K::NBW];
#pragma unroll
  for (int u = 0; u < K::NBW; ++u) {
    const int n0 = 16 * (grp * K::NBW + u) + lr, nn = n0 < K::NK ? n0 : K::NK - 1, c = nn / 7, j = nn - 7 * c;
    bp[u] = Qs + (K::S == 2 ? (2 * c + ((1 + j) & 1)) * K::QP + (1 + j) / 2 : c * K::QP + 1 + j) + 4 * lk;
  }
  f32x4 acc[K::MA][K::NBW];
#pragma unroll
  for (int m = 0; m < K::MA; ++m)
#pragma unroll
    for (int u = 0; u < K::NBW; ++u) acc[m][u] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int G = gridDim.x;
  const int c0 = (int)((int64_t)p.nchunk * blockIdx.x / G), c1 = (int)((int64_t)p.nchunk * (blockIdx.x + 1) / G);
  if (c0 < c1) fetch(c0);
  for (int chunk = c0; chunk < c1; ++chunk) {
    __syncthreads();  // the constants are there; the previous chunk's reads are done
    stage(chunk);
    __syncthreads();
    if (chunk + 1 < c1) fetch(chunk + 1);  // in flight during this chunk's MFMAs
#pragma unroll 1
    for (int ks = slice; ks < K::KC; ks += K::NS) {
      float4 av[K::MA];
#pragma unroll
      for (int m = 0; m < K::MA; ++m) av[m] = *reinterpret_cast<const float4*>(ap + m * 16 * K::PS + 16 * ks);
#pragma unroll
      for (int u = 0; u < K::NBW; ++u) {
        if (K::NGR > 1 && grp * K::NBW + u >= K::NB) break;  // wave-uniform
        float bv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[e] = bp[u][16 * ks + e];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int m = 0; m < K::MA; ++m)
            acc[m][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&av[m])[e], bv[e],
                                                             acc[m][u], 0, 0, 0);
      }
    }
  }
  // the slices' sums, a fixed tree: the upper half hands over to the lower
  for (int h = K::NS / 2; h >= 1; h >>= 1) {
    __syncthreads();
    if (slice >= h && slice < 2 * h) {
      f32x4* d = reinterpret_cast<f32x4*>(lds) + ((slice - h) * K::NGR + grp) * K::MA * K::NBW * 64 + lane;
#pragma unroll
      for (int m = 0; m < K::MA; ++m)
#pragma unroll
        for (int u = 0; u < K::NBW; ++u) d[(m * K::NBW + u) * 64] = acc[m][u];
    }
    __syncthreads();
    if (slice < h) {
      const f32x4* d = reinterpret_cast<const f32x4*>(lds) + (slice * K::NGR + grp) * K::MA * K::NBW * 64 + lane;
#pragma unroll
      for (int m = 0; m < K::MA; ++m)
#pragma unroll
        for (int u = 0; u < K::NBW; ++u) acc[m][u] += d[(m * K::NBW + u) * 64];
    }
  }
  if (slice > 0) return;
  // D[row = 4 lk + r][col = lr]: weight (a, n)
  float* out = p.partial + (int64_t)blockIdx.x * (K::CA * K::NK);
#pragma unroll
  for (int m = 0; m < K::MA; ++m)
#pragma unroll
    for (int u = 0; u < K::NBW; ++u) {
      const int nn = 16 * (grp * K::NBW + u) + lr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * m + 4 * lk + r;
        if (a < K::CA && nn < K::NK) out[a * K::NK + nn] = acc[m][u][r];
      }
    }
}

// Sum of every layer's partials, one launch: a block takes 64 weights of one
// layer, its four waves a quarter of the partials each (in order), FP64.
__global__ __launch_bounds__(256) void wgrad2_reduce(Wg2Tab t) {
  __shared__ double s[4][64];
  int blk = blockIdx.x, l = 0;
  while (blk >= t.e[l].blocks) blk -= t.e[l++].blocks;
  const Wg2Red& q = t.e[l];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, e = blk * 64 + lane;
  const int g0 = q.G * wave / 4, g1 = q.G * (wave + 1) / 4;
  double acc = 0.0;
  if (e < q.nw) {
    int g = g0;
    for (; g + 16 <= g1; g += 16) {
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = q.partial[(int64_t)(g + j) * q.nw + e];
#pragma unroll
      for (int j = 0; j < 16; ++j) acc += (double)v[j];
    }
    for (; g < g1; ++g) acc += (double)q.partial[(int64_t)g * q.nw + e];
  }
  s[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && e < q.nw) q.dw[e] = (float)(((s[0][lane] + s[1][lane]) + s[2][lane]) + s[3][lane]);
}

namespace wg2 {
// per layer of the reference network; chunks of about 35 KB, two blocks per CU
// (one of 16 waves for the 64-channel layers, whose partials are the largest)
typedef Cfg<8, 21, 2, 128, 8, DZ, RAW> L0;
typedef Cfg<16, 8, 2, 256, 8, DZ, ACT> L1;
typedef Cfg<32, 16, 2, 128, 8, DZ, ACT> L2;
typedef Cfg<64, 32, 2, 64, 16, DZ, ACT> L3;
typedef Cfg<64, 32, 2, 64, 16, ACT, DZ> L4;
typedef Cfg<32, 16, 2, 128, 8, ACT, DZ> L5;
typedef Cfg<16, 8, 2, 256, 8, ACT, DZ> L6;
typedef Cfg<8, 8, 2, 256, 8, ACT, DZ> L7;
typedef Cfg<1, 8, 1, 512, 8, RAW, ACT> L8;

template <class K>
int blocks(int n, int Lp) {
  const int64_t chunks = (int64_t)n * ((Lp + K::WT - 1) / K::WT);
  return (int)std::min<int64_t>(chunks, K::NW == 16 ? 256 : 512);
}

template <class K>
hipError_t launch(const Wg2Args& a, Wg2Red* red, hipStream_t st) {
  P2 p{};
  p.p = {a.p, a.pbn};
  p.q = {a.q, a.qbn};
  p.n = a.n;
  p.Lp = a.Lp;
  p.Lq = a.Lq;
  p.tchunks = (a.Lp + K::WT - 1) / K::WT;
  const int64_t chunks = (int64_t)a.n * p.tchunks;
  if (chunks > (int64_t)1 << 30) return hipErrorInvalidValue;
  p.nchunk = (int)chunks;
  p.partial = a.partial;
  const int G = blocks<K>(a.n, a.Lp);
  hipLaunchKernelGGL(wgrad2<K>, dim3(G), dim3(K::NTHR), 0, st, p);
  *red = {a.partial, a.dw, K::CA * K::NK, G, (K::CA * K::NK + 63) / 64};
  return hipGetLastError();
}
}  // namespace wg2

#define GW_WG2(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

size_t wgrad2_partial_floats(int l, int n, int Lp) {
  switch (l) {
#define GW_CASE(i) \
  case i: return (size_t)wg2::blocks<wg2::L##i>(n, Lp) * (wg2::L##i::CA * wg2::L##i::NK);
    GW_WG2(GW_CASE)
#undef GW_CASE
    default: return 0;
  }
}

hipError_t launch_wgrad2(int l, const Wg2Args& a, Wg2Red* red, hipStream_t st) {
  switch (l) {
#define GW_CASE(i) \
  case i: return wg2::launch<wg2::L##i>(a, red, st);
    GW_WG2(GW_CASE)
#undef GW_CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_wgrad2_reduce(const Wg2Tab& t, hipStream_t st) {
  int blocks = 0;
  for (int l = 0; l < t.n; ++l) blocks += t.e[l].blocks;
  hipLaunchKernelGGL(wgrad2_reduce, dim3(blocks), dim3(256), 0, st, t);
  return hipGetLastError();
}

}  // namespace gw
