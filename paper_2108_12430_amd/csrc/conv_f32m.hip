// FP32 1-D convolutions on the matrix cores: an implicit GEMM on
// v_mfma_f32_16x16x4_f32 (exact FP32 products, FP32 accumulation).
//
//   D[o][c] = sum_kappa A[o][kappa] B[kappa][c],  kappa = tap * CIP + channel
//
// with the column view of the BF16 kernels (make_geo: column c is output c of
// a conv, or input position m of a stride-2 transposed conv, whose outputs 2m
// and 2m + 1 are two phases of four taps).  CIP is C_in rounded up to a
// multiple of 4, so that one lane's 16-byte LDS read is four consecutive
// channels of one tap.  A K step takes 16 kappa: lane l holds kappa = 16 ks +
// 4 (l / 16) + e in element e of its 16-byte fragments, and four MFMAs take
// the elements in turn (MFMA e: A[row = l % 16][k = l / 16], B[k = l / 16]
// [col = l % 16], D[row = 4 (l / 16) + r][col = l % 16]).
//
// What bounds it: the matrix cores where C_in C_out is large (154 TFLOP/s is
// what a large FP32 product reaches here), HBM for the thin layers.  The
// direct kernels (conv_fp32.hip) read every input value from L1/L2 once per
// tap and pay one 4-byte load per 8 FMAs; here a value is read from HBM once
// per block, transposed into LDS, and each 16-byte LDS read feeds MTB * NPH
// groups of four MFMAs.  Measured, direct -> this kernel: the forward,
// recomputed and adjoint convolutions of a training step (batch 32 x 21 x
// 32768) 2090 -> 535 us (with the normalisations, their statistics and tanh
// inside, which were another 500 us); BBHnet FP32, 64 windows of 2 x 2048 (9.9
// GFLOP), 987 -> 147 us a call.  There the 128-channel convolution keeps the
// matrix cores 57% busy; the rest is the staging of a tile, which all of the two
// blocks a CU holds do at the same time, and the epilogue.
#include "train_epi.h"

namespace gw {

namespace f32m {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int cip4(int c) { return (c + 3) / 4 * 4; }
// LDS row stride (floats): an odd multiple of 16 bytes, so that the 16-byte
// reads of consecutive rows by consecutive lanes fall on distinct banks
constexpr int rs(int cip) { return (cip / 4) % 2 ? cip : cip + 4; }

}  // namespace f32m

// ---------------------------------------------------------------------------
// Weight fragments: (phase, channel tile, K step, lane, element).  One launch
// packs every layer of a network (the layers' tables ride in the arguments).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_f32m_kernel(F32PackTab t) {
  int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int l = 0;
  while (l < t.n && idx >= t.e[l].total) idx -= t.e[l++].total;
  if (l == t.n) return;
  const F32Pack& q = t.e[l];
  const int e = (int)(idx & 3), lane = (int)(idx >> 2) & 63;
  int f = (int)(idx >> 8);
  const int ks = f % q.KS;
  f /= q.KS;
  const int mt = f % q.MT, ph = f / q.MT;
  const int o = 16 * mt + (lane & 15), kappa = 16 * ks + 4 * (lane >> 4) + e;
  const int jj = kappa / q.cip, i = kappa - jj * q.cip;
  // conv: tap jj; transposed: input offset d = jj - padc of phase ph is tap ph + pad - s d
  const int j = q.tr ? ph + q.pad - q.s * (jj - q.padc) : jj;
  const bool on = o < q.Co && i < q.Ci && jj < q.kt && j >= 0 && j < q.k;
  q.out[idx] = on ? q.w[o * q.wso + i * q.wsi + j] : 0.0f;
}

F32Pack f32m_pack_entry(const float* w, int64_t wso, int64_t wsi, float* out, int Ci, int Co, int k, int s, int pad,
                        bool tr) {
  const Geo g = make_geo(tr, k, s, pad, 1 << 20);
  F32Pack q{};
  q.w = w;
  q.wso = wso;
  q.wsi = wsi;
  q.out = out;
  q.Ci = Ci;
  q.Co = Co;
  q.k = k;
  q.s = s;
  q.pad = pad;
  q.tr = tr ? 1 : 0;
  q.padc = g.padc;
  q.kt = g.kt;
  q.cip = f32m::cip4(Ci);
  q.MT = (Co + 15) / 16;
  q.KS = (g.kt * q.cip + 15) / 16;
  q.total = (int64_t)g.nph * q.MT * q.KS * 256;
  return q;
}

size_t f32m_packed_floats(int Ci, int Co, int k, int s, int pad, bool tr) {
  return (size_t)f32m_pack_entry(nullptr, 0, 0, nullptr, Ci, Co, k, s, pad, tr).total;
}

hipError_t launch_pack_f32m(const F32PackTab& t, hipStream_t st) {
  int64_t total = 0;
  for (int l = 0; l < t.n; ++l) total += t.e[l].total;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_f32m_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, t);
  return hipGetLastError();
}

// Stage ROWS input rows of a tile into LDS, [row][channel] with row stride
// RS; row r holds input position q0 + r * STEP (zero outside [0, Lin) and for
// channels past Ci).  STEP 1: an item is (four channels, four positions), four
// 16-byte loads transposed in registers into four 16-byte stores; with HALF
// > 0 row r goes to (r & 1) * HALF + r / 2, so that a stride-2 reader walks
// consecutive LDS rows.  STEP 2 (the residual shortcut's rows): the even
// positions of the same loads, q0 a multiple of 8.  Lanes take consecutive
// positions of one channel group, so the loads are coalesced; vec tells that
// every row of the input (and of z2) starts 16-byte aligned.  PRO transforms
// the samples on the way (never the padding): cb holds the channels' constants
// in LDS, [6][CIP] (mean, invstd, gamma, beta or gamma invstd, s1, s2), z2 the
// second operand of PRO_DZ.
template <int CIP, int ROWS, int RS, int HALF, int STEP, int PRO>
__device__ __forceinline__ void f32m_stage(float* tile, const float* x, const float* z2, const float* cb, int Ci,
                                           int Lin, int q0, bool vec, int tid) {
  constexpr int G = CIP / 4;
  constexpr int RPC = 4 / STEP;                         // rows per chunk of four positions
  constexpr int NCH = STEP == 1 ? (ROWS + 3 + 3) / 4 : ROWS / RPC;
  const int qa = q0 & ~3;                               // floor to a multiple of 4 (q0 may be negative)
  const int off = q0 - qa;                              // STEP 2: always 0
  constexpr int ITEMS = (NCH * G + 255) / 256, BM = PRO == PRO_DZ ? 2 : 6, BATCH = ITEMS < BM ? ITEMS : BM;
#pragma unroll 1
  for (int i0 = 0; i0 < ITEMS; i0 += BATCH) {
    float4 v[BATCH][4], z[PRO == PRO_DZ ? BATCH : 1][4];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int e = tid + 256 * (i0 + u), g = e / NCH, ch = e - g * NCH, q = qa + 4 * ch;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = 4 * g + k;
        v[u][k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (PRO == PRO_DZ) z[u][k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (g < G && i < Ci) {
          const int64_t o = (int64_t)i * Lin;
          if (vec && q >= 0 && q + 4 <= Lin) {
            v[u][k] = *reinterpret_cast<const float4*>(x + o + q);
            if (PRO == PRO_DZ) z[u][k] = *reinterpret_cast<const float4*>(z2 + o + q);
          } else {
            float* d = &v[u][k].x;
            float* dz = &z[PRO == PRO_DZ ? u : 0][k].x;
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (q + j >= 0 && q + j < Lin) {
                d[j] = x[o + q + j];
                if (PRO == PRO_DZ) dz[j] = z2[o + q + j];
              }
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int e = tid + 256 * (i0 + u), g = e / NCH, ch = e - g * NCH;
      if (g >= G) continue;
      if (PRO != PRO_NONE) {
        const int q = qa + 4 * ch;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float* c = cb + 4 * g + k;
          const float m = c[0], is = c[CIP], ga = c[2 * CIP], be = c[3 * CIP];
          float* d = &v[u][k].x;
          const float* dz = &z[PRO == PRO_DZ ? u : 0][k].x;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool live = 4 * g + k < Ci && q + j >= 0 && q + j < Lin;
            const float t = PRO == PRO_ACT ? bn_tanh_one(d[j], m, is, ga, be)
                                           : bn_dz_one(d[j], dz[j], m, is, be, c[4 * CIP], c[5 * CIP]);
            d[j] = live ? t : 0.0f;
          }
        }
      }
      const float4 p[4] = {make_float4(v[u][0].x, v[u][1].x, v[u][2].x, v[u][3].x),
                           make_float4(v[u][0].y, v[u][1].y, v[u][2].y, v[u][3].y),
                           make_float4(v[u][0].z, v[u][1].z, v[u][2].z, v[u][3].z),
                           make_float4(v[u][0].w, v[u][1].w, v[u][2].w, v[u][3].w)};
#pragma unroll
      for (int k = 0; k < RPC; ++k) {
        const int r = RPC * ch + k - (STEP == 1 ? off : 0);
        const int pr = HALF ? (r & 1) * HALF + (r >> 1) : r;
        if (r >= 0 && r < ROWS) *reinterpret_cast<float4*>(tile + pr * RS + 4 * g) = p[k * STEP];
      }
    }
  }
}

// The channels' constants of a PRO transform, to LDS
template <int CIP, int PRO>
__device__ __forceinline__ void f32m_consts(float* cb, const BnBwdP& q, int Ci, int tid) {
  if (tid >= CIP) return;
  const int c = tid < Ci ? tid : Ci - 1;
  const float is = q.bn.invstd[c], g = q.bn.gamma[c];
  cb[tid] = q.bn.mean[c];
  cb[CIP + tid] = is;
  cb[2 * CIP + tid] = g;
  cb[3 * CIP + tid] = PRO == PRO_DZ ? g * is : q.bn.beta[c];
  if (PRO == PRO_DZ) {
    cb[4 * CIP + tid] = q.sum_dh[c] * q.invN;
    cb[5 * CIP + tid] = q.sum_dhx[c] * q.invN;
  }
}

// One K step: NTW column tiles x NA A fragments, four MFMAs each, for the
// fragments from m0 on (a transposed layer's phase 0 has no fourth tap).
template <int NA, int NTW>
__device__ __forceinline__ void f32m_step(const float4 (&a)[NA], const float4 (&b)[NTW], f32m::f32x4 (&acc)[NTW][NA],
                                          int m0 = 0, int m1 = NA) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int m = 0; m < NA; ++m)
        if (m >= m0 && m < m1)
          acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&a[m])[e],
                                                           reinterpret_cast<const float*>(&b[t])[e], acc[t][m], 0, 0,
                                                           0);
}

// The convolution: a block computes columns [64 NTW ct, 64 NTW (ct + 1)) of
// channel tiles [MTB ms, MTB (ms + 1)) of window b (block (b MS + ms) tiles +
// ct, so that blocks in flight together read neighbouring inputs); wave w
// takes NTW column tiles and all of the block's channel tiles.  CSP > 0: the
// residual stage's 1x1 stride-2 shortcut, added to the same accumulators as
// further K steps from a second tile staged over the first.  Every output is
// the same sequence of operations whatever the tile, the split and the batch.
template <int CIP, int MTB, int NPH, int KT, int SC, int NTW, int EPI, int CSP, int PRO>
__global__ __launch_bounds__(256) void conv_f32m(ConvP p, F32Frags fr, F32Train tr, int padc, int ncol, int MT) {
  using namespace f32m;
  constexpr int TN = 64 * NTW;
  constexpr int ROWS = SC * (TN - 1) + KT;
  constexpr int RS = rs(CIP);
  constexpr int HALF = SC == 2 ? (ROWS + 1) / 2 : 0;
  constexpr int KS = (KT * CIP + 15) / 16;
  constexpr int NA = NPH * MTB;
  constexpr int RSX = CSP ? rs(CSP) : 4, KSX = CSP ? (CSP + 15) / 16 : 0;
  constexpr bool SUMS = EPI == EPI_STATS || EPI == EPI_BNBWD;
  constexpr int TIN = (HALF ? 2 * HALF : ROWS) * RS, TOUT = SUMS ? train_tile_floats(16 * MTB, TN * NPH) : 0;
  constexpr int TILE = TIN > TOUT ? TIN : TOUT;
  static_assert(CSP == 0 || (SC == 1 && NPH == 1 && TN * RSX <= TILE), "the shortcut's tile reuses the input's");
  __shared__ __attribute__((aligned(16))) float tile[TILE];
  __shared__ double wsum[4];
  __shared__ float cb[PRO == PRO_NONE ? 1 : 6 * CIP];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & 15, lg = lane >> 4;
  const int MS = MT / MTB, tiles = (ncol + TN - 1) / TN;
  const int ct = (int)(blockIdx.x % tiles), bm = (int)(blockIdx.x / tiles), b = bm / MS, ms = bm - b * MS;
  const int col0 = ct * TN;
  const float* xb = p.x + (int64_t)b * p.Ci * p.Lin;
  if (PRO != PRO_NONE) {
    f32m_consts<CIP, PRO>(cb, tr.in, p.Ci, tid);
    __syncthreads();
  }
  f32m_stage<CIP, ROWS, RS, HALF, 1, PRO>(
      tile, xb, PRO == PRO_DZ ? tr.in.z + (int64_t)b * p.Ci * p.Lin : nullptr, cb, p.Ci, p.Lin, SC * col0 - padc,
      ((p.Lin & 3) | (reinterpret_cast<uintptr_t>(p.x) & 15) |
       (PRO == PRO_DZ ? reinterpret_cast<uintptr_t>(tr.in.z) & 15 : 0)) == 0,
      tid);
  // A fragments of phase ph, channel tile ms MTB + m: two K steps requested ahead
  const float4* wp = reinterpret_cast<const float4*>(fr.w) + (int64_t)ms * MTB * KS * 64 + lane;
  auto frag = [&](int m, int ks) {  // m = ph MTB + channel tile
    return wp[((int64_t)(m / MTB) * MT + m % MTB) * KS * 64 + ks * 64];
  };
  float4 a0[NA], a1[NA];
#pragma unroll
  for (int m = 0; m < NA; ++m) {
    a0[m] = frag(m, 0);
    a1[m] = frag(m, KS > 1 ? 1 : 0);
  }
  f32x4 acc[NTW][NA];
#pragma unroll
  for (int t = 0; t < NTW; ++t)
#pragma unroll
    for (int m = 0; m < NA; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  const float* colbase = tile + (wave * NTW * 16 + lc) * RS;
  // B fragments of K step ks.  K entries past the last tap are zeros, never a
  // real sample under a zero weight: an infinite sample must not reach an
  // output that does not read it.
  auto bfrag = [&](int ks, float4 (&bv)[NTW]) {
    const int kappa = 16 * ks + 4 * lg, j0 = kappa / CIP, i0 = kappa - j0 * CIP;
    const int jj = j0 < KT ? j0 : KT - 1;
    const int row = SC == 2 ? (jj & 1) * HALF + (jj >> 1) : jj;
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      bv[t] = *reinterpret_cast<const float4*>(colbase + (row + 16 * t) * RS + i0);
      if (16 * ks + 16 > KT * CIP && j0 >= KT) bv[t] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  // the MFMAs of K step ks; for the same reason a transposed layer's phase 0,
  // which has three taps, leaves out its fourth input offset
  auto step = [&](int ks, const float4 (&a)[NA], const float4 (&bv)[NTW]) {
    if (NPH == 2 && 16 * ks + 16 > 3 * CIP) {
      f32m_step<NA, NTW>(a, bv, acc, MTB, NA);  // phase 1
      if (16 * ks < 3 * CIP) {                  // the step straddles the offsets
        float4 bz[NTW];
#pragma unroll
        for (int t = 0; t < NTW; ++t) bz[t] = 16 * ks + 4 * lg < 3 * CIP ? bv[t] : make_float4(0.f, 0.f, 0.f, 0.f);
        f32m_step<NA, NTW>(a, bz, acc, 0, MTB);
      }
    } else {
      f32m_step<NA, NTW>(a, bv, acc);
    }
  };
  constexpr int KSE = KS & ~1, KU = KS <= 16 ? 8 : 2;
#pragma unroll KU
  for (int ks = 0; ks < KSE; ks += 2) {
    float4 bv[NTW];
    bfrag(ks, bv);
    step(ks, a0, bv);
#pragma unroll
    for (int m = 0; m < NA; ++m) a0[m] = frag(m, ks + 2 < KS ? ks + 2 : KS - 1);
    bfrag(ks + 1, bv);
    step(ks + 1, a1, bv);
#pragma unroll
    for (int m = 0; m < NA; ++m) a1[m] = frag(m, ks + 3 < KS ? ks + 3 : KS - 1);
  }
  if constexpr (KS & 1) {
    float4 bv[NTW];
    bfrag(KS - 1, bv);
    step(KS - 1, a0, bv);
  }
  if constexpr (CSP > 0) {
    __syncthreads();  // every wave is done reading the input tile
    const float* xs = p.xs + (int64_t)b * p.Cs * p.Ls;
    f32m_stage<CSP, TN, RSX, 0, 2, PRO_NONE>(tile, xs, nullptr, nullptr, p.Cs, p.Ls, 2 * col0,
                                             (p.Ls & 3) == 0 && (reinterpret_cast<uintptr_t>(p.xs) & 15) == 0, tid);
    __syncthreads();
    const float4* sp = reinterpret_cast<const float4*>(fr.ws) + (int64_t)ms * MTB * KSX * 64 + lane;
#pragma unroll
    for (int ks = 0; ks < KSX; ++ks) {
      const int kappa = 16 * ks + 4 * lg, i0 = kappa < CSP ? kappa : 0;
      float4 av[NA], bv[NTW];
#pragma unroll
      for (int m = 0; m < NA; ++m) av[m] = sp[(m * KSX + ks) * 64];
#pragma unroll
      for (int t = 0; t < NTW; ++t) {
        bv[t] = *reinterpret_cast<const float4*>(tile + ((wave * NTW + t) * 16 + lc) * RSX + i0);
        if (16 * KSX > CSP && kappa >= CSP) bv[t] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      f32m_step<NA, NTW>(av, bv, acc);
    }
  }
  if constexpr (SUMS) {
    train_epilogue<MTB, NPH, NTW, EPI>(p, tr, acc, tile, b, col0, b * tiles + ct, (int)gridDim.x, tid);
    return;
  }
  // epilogue: lane (lc, lg) holds channels 16 mt + 4 lg + r of column c
  double gsum = 0.0;  // FP64: the pooled head's terms cancel
#pragma unroll
  for (int m = 0; m < MTB; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 16 * (ms * MTB + m) + 4 * lg + r;
      if (o >= p.Co) continue;
      float kb = 0.0f, ka = 1.0f;
      if (EPI == EPI_OUT) {
        ka = p.scale[o];
        kb = p.shift[o];
      } else if (EPI == EPI_RESID_RELU || EPI == EPI_RESID_GAP) {
        kb = p.bias[o] + p.bs[o];
        if (EPI == EPI_RESID_GAP) ka = p.hw[o];
      } else if (p.bias) {
        kb = p.bias[o];
      }
#pragma unroll
      for (int t = 0; t < NTW; ++t) {
        const int col = col0 + (wave * NTW + t) * 16 + lc;
        if (col >= ncol) continue;
        if constexpr (NPH == 2) {
          const float2 v = make_float2(acc[t][m][r] + kb, acc[t][MTB + m][r] + kb);
          float* y = p.y + ((int64_t)b * p.Co + o) * p.Lout + 2 * col;
          if (2 * col + 1 < p.Lout) {
            if (((p.Lout & 1) | (reinterpret_cast<uintptr_t>(p.y) & 7)) == 0) {
              *reinterpret_cast<float2*>(y) = v;
            } else {
              y[0] = v.x;
              y[1] = v.y;
            }
          } else {
            y[0] = v.x;
          }
        } else if constexpr (EPI == EPI_OUT) {
          const int W = p.Lout;
          const float v = fmaf(acc[t][m][r], ka, kb);
          if (p.noise) p.noise[(int64_t)b * W + col] = v;
          if (p.clean) {
            const Item& it = p.items[b];
            const int t0 = W - it.s - it.delay;
            if (col >= t0 && col < t0 + it.s) {
              const int64_t idx = it.out + (col - t0);
              p.clean[idx] = p.strain[idx] - v;
            }
          }
        } else if constexpr (EPI == EPI_RESID_GAP) {
          gsum += (double)ka * (double)fmaxf(acc[t][m][r] + kb, 0.0f);
        } else {
          float v = acc[t][m][r] + kb;
          if (EPI != EPI_BIAS) v = fmaxf(v, 0.0f);
          p.y[((int64_t)b * p.Co + o) * p.Lout + col] = v;
        }
      }
    }
  if constexpr (EPI == EPI_RESID_GAP) {
    // fixed-order reduction: lanes of a wave, then the four waves
    for (int off = 32; off > 0; off >>= 1) gsum += __shfl_down(gsum, off, 64);
    if (lane == 0) wsum[wave] = gsum;
    __syncthreads();
    if (tid == 0)
      fr.gap_part[((int64_t)b * tiles + ct) * MS + ms] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
  }
}

// Compiled shapes: (CIP, MT, NPH, KT, SC, EPI, CSP) with the block's channel
// tiles MTB and column tiles per wave NTW: at most eight accumulator tiles a
// wave, so that two to four blocks share a CU and one block's staging runs
// under another's MFMAs.
#define GW_F32M_SHAPES(X)                                                            \
  /* DeepClean training: forward and adjoint convolutions, output conv */            \
  X(24, 1, 1, 7, 2, EPI_BIAS, 0, 1, 4, PRO_NONE) \
  X(8, 1, 1, 7, 2, EPI_BIAS, 0, 1, 4, PRO_NONE) \
  X(16, 2, 1, 7, 2, EPI_BIAS, 0, 2, 2, PRO_NONE) \
  X(32, 4, 1, 7, 2, EPI_BIAS, 0, 4, 2, PRO_NONE) \
  X(64, 2, 2, 4, 1, EPI_BIAS, 0, 2, 2, PRO_NONE) \
  X(32, 1, 2, 4, 1, EPI_BIAS, 0, 1, 4, PRO_NONE) \
  X(16, 1, 2, 4, 1, EPI_BIAS, 0, 1, 4, PRO_NONE) \
  X(8, 1, 2, 4, 1, EPI_BIAS, 0, 1, 4, PRO_NONE) \
  X(4, 1, 1, 7, 1, EPI_BIAS, 0, 1, 4, PRO_NONE) \
  X(8, 1, 1, 7, 1, EPI_OUT, 0, 1, 4, PRO_NONE) \
  /* BBHnet stages */                                                                \
  X(4, 2, 1, 7, 2, EPI_RELU, 0, 2, 2, PRO_NONE) \
  X(32, 2, 1, 7, 1, EPI_RESID_RELU, 4, 2, 2, PRO_NONE) \
  X(32, 4, 1, 7, 2, EPI_RELU, 0, 2, 2, PRO_NONE) \
  X(64, 4, 1, 7, 1, EPI_RESID_RELU, 32, 2, 2, PRO_NONE) \
  X(64, 8, 1, 7, 2, EPI_RELU, 0, 2, 2, PRO_NONE) \
  X(128, 8, 1, 7, 1, EPI_RESID_RELU, 64, 2, 2, PRO_NONE) \
  X(128, 8, 1, 7, 1, EPI_RESID_GAP, 64, 2, 2, PRO_NONE) \
  /* DeepClean training, the reference network: activations taken from z as   \
     they are staged, statistics in the epilogue; adjoint convolutions whose  \
     input is dz and whose output is the next layer's dh */                   \
  X(24, 1, 1, 7, 2, EPI_STATS, 0, 1, 2, PRO_NONE) \
  X(8, 1, 1, 7, 2, EPI_STATS, 0, 1, 4, PRO_ACT) \
  X(16, 2, 1, 7, 2, EPI_STATS, 0, 2, 2, PRO_ACT) \
  X(32, 4, 1, 7, 2, EPI_STATS, 0, 4, 2, PRO_ACT) \
  X(64, 2, 2, 4, 1, EPI_STATS, 0, 2, 1, PRO_ACT) \
  X(32, 1, 2, 4, 1, EPI_STATS, 0, 1, 2, PRO_ACT) \
  X(16, 1, 2, 4, 1, EPI_STATS, 0, 1, 4, PRO_ACT) \
  X(8, 1, 2, 4, 1, EPI_STATS, 0, 1, 4, PRO_ACT) \
  X(8, 1, 1, 7, 1, EPI_OUT, 0, 1, 4, PRO_ACT) \
  X(4, 1, 1, 7, 1, EPI_BNBWD, 0, 1, 4, PRO_NONE) \
  X(8, 1, 1, 7, 2, EPI_BNBWD, 0, 1, 4, PRO_DZ) \
  X(16, 2, 1, 7, 2, EPI_BNBWD, 0, 2, 2, PRO_DZ) \
  X(32, 4, 1, 7, 2, EPI_BNBWD, 0, 4, 2, PRO_DZ) \
  X(64, 2, 2, 4, 1, EPI_BNBWD, 0, 2, 2, PRO_DZ) \
  X(32, 1, 2, 4, 1, EPI_BNBWD, 0, 1, 4, PRO_DZ) \
  X(16, 1, 2, 4, 1, EPI_BNBWD, 0, 1, 4, PRO_DZ)

template <int CIP, int MT, int NPH, int KT, int SC, int EPI, int CSP, int MTB, int NTW, int PRO>
static hipError_t launch_f32m_t(const ConvP& p, const F32Frags& f, const F32Train& t, const Geo& g, hipStream_t st) {
  const int64_t blocks = (int64_t)p.n * (MT / MTB) * ((g.ncol + 64 * NTW - 1) / (64 * NTW));
  if (blocks > ((int64_t)1 << 31) - 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL((conv_f32m<CIP, MTB, NPH, KT, SC, NTW, EPI, CSP, PRO>), dim3((unsigned)blocks), dim3(256), 0, st, p, f, t,
                     g.padc, g.ncol, MT);
  return hipGetLastError();
}

bool conv_f32m_supported(int Ci, int Co, int k, int s, int pad, bool tr, int epi, int Cs, int pro) {
  if (k != 7 || pad != 3 || (tr && s != 1 && s != 2)) return false;
  const Geo g = make_geo(tr, k, s, pad, 1 << 20);
  const int cip = f32m::cip4(Ci), mt = (Co + 15) / 16, csp = Cs ? f32m::cip4(Cs) : 0;
#define GW_SUP(CIP, MT, NPH, KT, SC, EPI, CSP, MTB, NTW, PRO)                                                         \
  if (cip == CIP && mt == MT && g.nph == NPH && g.kt == KT && g.sc == SC && epi == EPI && csp == CSP && pro == PRO) \
    return true;
  GW_F32M_SHAPES(GW_SUP)
#undef GW_SUP
  return false;
}

int conv_f32m_gap_parts(int Co, int Lout) {
  return (Lout + 127) / 128 * ((Co + 15) / 16 / 2);  // the pooled variant's column tiles x channel shares
}

int conv_f32m_blocks(int Ci, int Co, int n, int Lout, int k, int s, int pad, bool tr, int epi) {
  const Geo g = make_geo(tr, k, s, pad, Lout);
  const int cip = f32m::cip4(Ci), mt = (Co + 15) / 16;
#define GW_BLK(CIP, MT, NPH, KT, SC, EPI, CSP, MTB, NTW, PRO)                                       \
  if (cip == CIP && mt == MT && g.nph == NPH && g.kt == KT && g.sc == SC &&                         \
      EPI == epi)                                                                                   \
    return n * ((g.ncol + 64 * NTW - 1) / (64 * NTW));
  GW_F32M_SHAPES(GW_BLK)
#undef GW_BLK
  return -1;
}

hipError_t launch_conv_f32m(const ConvP& p, const F32Frags& f, bool tr, int epi, hipStream_t st, int pro,
                            const F32Train* t) {
  const Geo g = make_geo(tr, p.k, p.stride, p.pad, p.Lout);
  const bool res = epi == EPI_RESID_RELU || epi == EPI_RESID_GAP;
  if (!f.w || !p.x || (res && (!f.ws || !p.xs || p.Ls != 2 * p.Lout))) return hipErrorInvalidValue;
  if (epi == EPI_RESID_GAP && (!p.hw || !f.gap_part)) return hipErrorInvalidValue;
  if (p.ldx && p.ldx != p.Lin) return hipErrorInvalidValue;
  const F32Train tt = t ? *t : F32Train{};
  if ((epi == EPI_STATS || epi == EPI_BNBWD) && (!tt.partial || !p.y)) return hipErrorInvalidValue;
  if ((epi == EPI_STATS || epi == EPI_BNBWD) && !train_epilogue_fits(p.Co, (p.Co + 15) / 16)) return hipErrorInvalidValue;
  if (epi == EPI_BNBWD && !tt.z) return hipErrorInvalidValue;
  if (pro == PRO_DZ && !tt.in.z) return hipErrorInvalidValue;
  const int cip = f32m::cip4(p.Ci), mt = (p.Co + 15) / 16, csp = res ? f32m::cip4(p.Cs) : 0;
#define GW_LAUNCH(CIP, MT, NPH, KT, SC, EPI, CSP, MTB, NTW, PRO)                                                       \
  if (cip == CIP && mt == MT && g.nph == NPH && g.kt == KT && g.sc == SC && epi == EPI && csp == CSP && pro == PRO &&  \
      p.k == 7 && p.pad == 3)                                                                                          \
    return launch_f32m_t<CIP, MT, NPH, KT, SC, EPI, CSP, MTB, NTW, PRO>(p, f, tt, g, st);
  GW_F32M_SHAPES(GW_LAUNCH)
#undef GW_LAUNCH
  return hipErrorNotSupported;
}

}  // namespace gw
