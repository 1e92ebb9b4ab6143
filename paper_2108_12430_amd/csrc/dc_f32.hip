// Fused FP32 DeepClean forward: one block computes T consecutive output
// samples of one window through all nine layers of the reference network,
// with every intermediate activation in LDS, on v_mfma_f32_16x16x4_f32 (exact
// FP32 products, FP32 accumulation).
//
// Working back from the output tile [u0, u0 + T), each layer's needed outputs
// are a fixed range around its scaled tile start (LO, NR below); positions
// outside a layer's signal are stored as zeros, the next layer's padding.  The
// order of operations behind an output does not depend on T, on the tile it
// falls in or on the batch, so every variant gives the same bits.
//
// Layouts.  The input tile is [channel][time] as the windows are, so staging
// is a plain copy; layer 0 takes K = channel x tap (eight taps, the eighth
// zero) and reads four consecutive samples a lane.  The activations are
// [time][channel] with row strides that are odd multiples of 16 bytes (even
// and odd rows apart where the reader steps two rows); K = tap x channel, and
// a lane's 16-byte read is four channels of one tap.  A K step takes 16 K
// entries in four MFMAs; its weight fragment is one 16-byte load a lane from
// L2, requested two steps ahead (the next layer's first two before the
// barrier between the layers).
//
// No output ever meets a sample outside its receptive field, not even under a
// zero weight (0 * inf is not 0): K entries past the taps take zeros, and a
// transposed layer's phase 0, which has three taps of the four input offsets,
// leaves the fourth out (the stacked layers 6 and 7 add it from accumulators
// of their own to phase 1's rows only).
//
// What bounds it: the matrix cores.  Per 512 samples the tile's padded GEMMs
// take 3450 MFMAs of 32 cycles, 11.5 us of a CU, so a 21 x 32768 window
// cannot take less than 2.9 us of the whole chip (1.7 us without tile and
// channel padding).  Measured, nine direct launches -> this kernel: one 21 x
// 4096 window 302 -> 17 us, 16 windows of 21 x 32768 475 -> 101 us (4.2
// GFLOP, 42 TFLOP/s).
#include "internal.h"

namespace gw {
namespace f32d {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NW = 8;  // waves per block
constexpr int NTHR = 64 * NW;
constexpr int C[10] = {21, 8, 16, 32, 64, 32, 16, 8, 8, 1};
constexpr int LO[10] = {-93, -45, -21, -9, -3, -3, -3, -3, -3, 0};
constexpr int RS(int l) { return C[l] % 8 ? C[l] : C[l] + 4; }  // activations: an odd multiple of 4 floats
constexpr bool STACK(int l) { return l == 6 || l == 7; }        // rows = 8 phase + channel
constexpr int MT(int l) { return (C[l + 1] + 15) / 16; }
constexpr int NPH(int l) { return l == 4 || l == 5 ? 2 : 1; }
constexpr int QP(int l) { return NPH(l) * MT(l); }  // (phase, channel tile) pairs
constexpr int KT(int l) { return l < 4 ? 7 : 4; }
constexpr int KS(int l) { return l == 0 ? 11 : (KT(l) * C[l] + 15) / 16; }
constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }
constexpr int mx(int a, int b) { return a > b ? a : b; }

template <int T>
struct G {
  static_assert(T % 128 == 0, "whole 16-position bottleneck steps");
  // needed rows of a_1 .. a_8 (row 0 at the scaled tile start + LO)
  static constexpr int NR(int l) {
    return l == 1 ? T / 2 + 91 : l == 2 ? T / 4 + 43 : l == 3 ? T / 8 + 19 : l == 4 ? T / 16 + 7 : l == 5 ? T / 8 + 7
         : l == 6 ? T / 4 + 7 : l == 7 ? T / 2 + 7 : T + 6;
  }
  // columns: one per output row (convs), one per input position (transposed:
  // column c makes rows 2c - 1 and 2c)
  static constexpr int NCOL(int l) {
    return l < 4 ? NR(l + 1) : l == 4 ? T / 16 + 4 : l == 5 ? T / 8 + 4 : l == 6 ? T / 4 + 4 : T / 2 + 4;
  }
  static constexpr int NT(int l) { return cdiv(NCOL(l), 16); }
  // column tiles per work unit (a unit: one (phase, channel tile) pair)
  static constexpr int NTC(int l) { return cdiv(NT(l) * QP(l), NW); }
  static constexpr int NG(int l) { return cdiv(NT(l), NTC(l)); }
  static constexpr int NU(int l) { return NG(l) * QP(l); }
  static constexpr int XW = 2 * (16 * NT(0) - 1) + 8;  // staged samples per channel
  // rows of layer l's input buffer its (padded) columns may read
  static constexpr int ROWS(int l) {
    return mx(l == 8 ? T + 6 : (l < 4 ? 2 : 1) * (16 * NT(l) - 1) + KT(l), NR(l));
  }
  static constexpr int HALF(int l) { return l >= 1 && l <= 3 ? (ROWS(l) + 1) / 2 : 0; }
  static constexpr int SZ(int l) { return l == 0 ? C[0] * XW : (HALF(l) ? 2 * HALF(l) : ROWS(l)) * RS(l); }
  // ping-pong: inputs of layers 0, 2, 4, 6, 8 in A, of 1, 3, 5, 7 in B
  static constexpr int BUFA = cdiv(mx(mx(mx(SZ(0), SZ(2)), mx(SZ(4), SZ(6))), SZ(8)), 4) * 4;
  static constexpr int BUFB = cdiv(mx(mx(SZ(1), SZ(3)), mx(SZ(5), SZ(7))), 4) * 4;
  __device__ static constexpr int prow(int l, int r) { return HALF(l) ? (r & 1) * HALF(l) + (r >> 1) : r; }
};

}  // namespace f32d

struct DcF32P {
  const float* wpk[9];
  const float* scale[9];
  const float* shift[9];
};

// Special fragments: layer 0 (K = channel x 8 taps), the stacked layers 6 and
// 7 (rows 8 phase + channel, K = input offset x channel) and layer 8's plain
// weights as [tap][channel].
__global__ __launch_bounds__(256) void pack_dc_f32_kernel(const float* w, float* out, int l, int total) {
  using namespace f32d;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  if (l == 8) {
    out[idx] = w[(idx % 8) * 7 + idx / 8];
    return;
  }
  const int e = idx & 3, lane = (idx >> 2) & 63, ks = idx >> 8, row = lane & 15;
  const int kappa = 16 * ks + 4 * (lane >> 4) + e;
  float v = 0.0f;
  if (l == 0) {
    const int ch = kappa >> 3, j = kappa & 7;
    if (row < 8 && ch < 21 && j < 7) v = w[(row * 21 + ch) * 7 + j];
  } else {
    const int ci = l == 6 ? 16 : 8, ph = row >> 3, o = row & 7, d = kappa / ci - 1, i = kappa % ci;
    const int j = ph + 3 - 2 * d;
    if (kappa < 4 * ci && j >= 0 && j < 7) v = w[(i * 8 + o) * 7 + j];
  }
  out[idx] = v;
}

// Which layers' fragments pack_dc_f32_kernel makes, and their floats; the
// others use the general FP32 fragments (launch_pack_f32m).
size_t dc_f32_special_floats(int l) {
  return l == 0 || l == 6 || l == 7 ? (size_t)f32d::KS(l) * 256 : l == 8 ? 56 : 0;
}

hipError_t launch_pack_dc_f32(const float* w, float* out, int l, hipStream_t st) {
  const int total = (int)dc_f32_special_floats(l);
  if (!total) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pack_dc_f32_kernel, dim3((total + 255) / 256), dim3(256), 0, st, w, out, l, total);
  return hipGetLastError();
}

// Stage a tile's input: samples [p0, p0 + XW) of every channel (zero outside
// [0, Lin)).  A thread takes one sample of every channel, so it computes one
// address and its 21 loads are in flight together, each coalesced over the
// wave; nothing is assumed of alignment, and a ring's wrap is one compare.
// UPD: the newest s samples come from the request (p.upd) and are written to
// the ring and its BF16 shadow on the way; tiles that share a sample write the
// same values, and no tile reads the ring positions they replace.
template <int T, int SRC, bool UPD>
__device__ __forceinline__ void f32d_stage(float* xt, const DcIn& p, int b, int p0, int tid) {
  using namespace f32d;
  constexpr int XW = G<T>::XW;
  const float* base;
  int ld, head = 0, snew = p.Lin, s = 0;
  uint16_t* sh = nullptr;
  const float* src = nullptr;
  if (SRC == SRC_RING) {
    const Item& it = p.items[b];
    base = reinterpret_cast<const float*>(p.arena) + it.ring;
    ld = it.W;
    head = it.head;
    if (UPD) {
      s = it.s;
      snew = p.Lin - s;
      sh = reinterpret_cast<uint16_t*>(const_cast<void*>(p.arena)) + it.shadow;
      src = p.upd + it.src;
    }
  } else {
    ld = p.ldx;
    base = p.x + (int64_t)b * C[0] * ld;
  }
#pragma unroll
  for (int k = 0; k < cdiv(XW, NTHR); ++k) {
    const int c = tid + k * NTHR, q = p0 + c;
    const bool live = c < XW && q >= 0 && q < p.Lin;
    int at = live ? q : 0;
    if (SRC == SRC_RING) {
      at += head;
      if (at >= ld) at -= ld;
    }
    const bool fresh = UPD && live && q >= snew;
    const float* from = fresh ? src + (q - snew) : base + at;
    const int64_t step = fresh ? s : ld;
    float v[C[0]];
#pragma unroll
    for (int i = 0; i < C[0]; ++i) v[i] = from[i * step];
    if (fresh) {
      float* ring = const_cast<float*>(base) + at;
#pragma unroll
      for (int i = 0; i < C[0]; ++i) {
        ring[(int64_t)i * ld] = v[i];
        sh[(int64_t)i * ld + at] = f2bf(v[i]);
      }
    }
    if (c < XW)
#pragma unroll
      for (int i = 0; i < C[0]; ++i) xt[i * XW + c] = live ? v[i] : 0.0f;
  }
}

// wave `wave`'s first two weight fragments of layer l
template <int T, int l>
__device__ __forceinline__ void f32d_first(float4 (&a)[2], const float* w, int wave, int lane) {
  using namespace f32d;
  if (l > 7 || wave >= G<T>::NU(l)) return;  // wave-uniform
  const float4* wq = reinterpret_cast<const float4*>(w) + (wave % QP(l)) * KS(l) * 64 + lane;
  a[0] = wq[0];
  a[1] = wq[64];
}

// BN + tanh of channels o0 .. o0 + 3 of output row `row`, one 16-byte store;
// zero outside the layer's signal.
template <int T, int l>
__device__ __forceinline__ void f32d_epi(float* out, int row, int o0, f32d::f32x4 v, const float4& sc, const float4& sh,
                                         int pos0, int Lout) {
  using namespace f32d;
  if (row < 0 || row >= G<T>::NR(l + 1)) return;
  const int u = pos0 + row;
  const bool live = u >= 0 && u < Lout;
  float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live) {
    t.x = tanhf(fmaf(v[0], sc.x, sh.x));
    t.y = tanhf(fmaf(v[1], sc.y, sh.y));
    t.z = tanhf(fmaf(v[2], sc.z, sh.z));
    t.w = tanhf(fmaf(v[3], sc.w, sh.w));
  }
  *reinterpret_cast<float4*>(out + G<T>::prow(l + 1, row) * RS(l + 1) + o0) = t;
}

// Layer l < 8: LDS in -> LDS out.  Unit u = (column group) x (pair q); wave w
// takes units w, w + NW, ...
template <int T, int l>
__device__ __forceinline__ void f32d_layer(int tid, const float* in, float* out, float4 (&af)[2], const float* w,
                                           const float* wn, const float* ksc, const float* ksh, int pos0, int Lout) {
  using namespace f32d;
  using g = G<T>;
  constexpr int CI = C[l], NTn = g::NT(l), NTCl = g::NTC(l), QPl = QP(l), KSn = KS(l);
  constexpr int STEP = l == 0 ? 2 : RS(l);  // floats between adjacent columns (split rows: adjacent LDS rows)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & 15, lg = lane >> 4;
#pragma unroll 1
  for (int unit = wave; unit < g::NU(l); unit += NW) {
    const int q = unit % QPl, nt0 = unit / QPl * NTCl;  // wave-uniform
    const int ph = q / MT(l), mt = q % MT(l);
    const float4* wq = reinterpret_cast<const float4*>(w) + q * KSn * 64 + lane;
    if (unit != wave) {
      af[0] = wq[0];
      af[1] = wq[64];
    }
    const float* colbase = in + (nt0 * 16 + lc) * STEP;
    // even and odd K steps of the longer sums add up apart (half the rounding
    // chain; the stacked layers' acc2: phase 1's fourth offset)
    f32x4 acc[NTCl], acc2[NTCl];
#pragma unroll
    for (int a = 0; a < NTCl; ++a) {
      acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
      acc2[a] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // tiles past the layer's last re-read that one (their sums are not stored)
    auto off = [&](int a) { return (a < NTn - nt0 ? a : NTn - 1 - nt0) * 16 * STEP; };
    auto bfrag = [&](int ks, float4 (&bv)[NTCl]) {
      if constexpr (l == 0) {
        const int ch = 2 * ks + (lg >> 1), i0 = (ch < CI ? ch : CI - 1) * g::XW + 4 * (lg & 1);
#pragma unroll
        for (int a = 0; a < NTCl; ++a) {
          const float2 u = *reinterpret_cast<const float2*>(colbase + i0 + off(a));
          const float2 v = *reinterpret_cast<const float2*>(colbase + i0 + off(a) + 2);
          bv[a] = make_float4(u.x, u.y, v.x, (lg & 1) ? 0.0f : v.y);  // no eighth tap
          if (ks == KSn - 1 && ch >= CI) bv[a] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      } else {
        const int kappa = 16 * ks + 4 * lg, j0 = kappa / CI, i0 = kappa - j0 * CI;
        const int jj = j0 < KT(l) ? j0 : KT(l) - 1;
        const int row = g::HALF(l) ? (jj & 1) * g::HALF(l) + (jj >> 1) : jj;
#pragma unroll
        for (int a = 0; a < NTCl; ++a) {
          bv[a] = *reinterpret_cast<const float4*>(colbase + row * RS(l) + i0 + off(a));
          if (16 * ks + 16 > KT(l) * CI && j0 >= KT(l)) bv[a] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
    };
    auto mma = [&](const float4& av, const float4 (&bv)[NTCl], f32x4 (&c)[NTCl]) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int a = 0; a < NTCl; ++a)
          c[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&av)[e],
                                                      reinterpret_cast<const float*>(&bv[a])[e], c[a], 0, 0, 0);
    };
    if constexpr (STACK(l)) {
      // offsets 0 .. 2 of the input go to both phases, offset 3 to phase 1
      float4 av[KSn];
#pragma unroll
      for (int ks = 0; ks < KSn; ++ks) av[ks] = ks < 2 ? af[ks] : wq[ks * 64];
#pragma unroll
      for (int ks = 0; ks < KSn; ++ks) {
        float4 bv[NTCl];
        bfrag(ks, bv);
        if (16 * ks + 16 <= 3 * CI) {
          mma(av[ks], bv, acc);
        } else if (16 * ks >= 3 * CI) {
          mma(av[ks], bv, acc2);
        } else {  // CI = 8: lane groups 0, 1 hold offset 2, groups 2, 3 offset 3
          const bool third = 16 * ks + 4 * lg >= 3 * CI;
          float4 b0[NTCl], b1[NTCl];
#pragma unroll
          for (int a = 0; a < NTCl; ++a) {
            b0[a] = third ? make_float4(0.f, 0.f, 0.f, 0.f) : bv[a];
            b1[a] = third ? bv[a] : make_float4(0.f, 0.f, 0.f, 0.f);
          }
          mma(av[ks], b0, acc);
          mma(av[ks], b1, acc2);
        }
      }
    } else {
      // phase 0 of a transposed layer stops before its fourth input offset
      const int kend = NPH(l) == 2 && ph == 0 ? 3 * CI / 16 : KSn;  // wave-uniform
      float4 a0 = af[0], a1 = af[1];
      constexpr int KU = KSn <= 11 ? 6 : 2;
#pragma unroll KU
      for (int ks = 0; ks + 1 < kend; ks += 2) {
        float4 bv[NTCl];
        bfrag(ks, bv);
        mma(a0, bv, acc);
        a0 = wq[(ks + 2 < KSn ? ks + 2 : KSn - 1) * 64];
        bfrag(ks + 1, bv);
        mma(a1, bv, acc2);
        a1 = wq[(ks + 3 < KSn ? ks + 3 : KSn - 1) * 64];
      }
      if constexpr (KSn % 2 == 1) {
        float4 bv[NTCl];
        bfrag(KSn - 1, bv);
        mma(a0, bv, acc);
      }
    }
    if (unit + NW >= g::NU(l)) f32d_first<T, l + 1>(af, wn, wave, lane);
    // epilogue: lane (lc, lg) holds rows 4 lg .. 4 lg + 3 of column nt0 16 + lc
    const int o0 = STACK(l) ? 4 * (lg & 1) : 16 * mt + 4 * lg;
    if (o0 < C[l + 1]) {
      const float4 sc = *reinterpret_cast<const float4*>(ksc + o0), sh = *reinterpret_cast<const float4*>(ksh + o0);
#pragma unroll
      for (int a = 0; a < NTCl; ++a) {
        if (nt0 + a >= NTn) break;
        const int c = (nt0 + a) * 16 + lc;
        if constexpr (STACK(l)) {
          f32x4 v = acc[a];
          if (lg >= 2) v += acc2[a];
          f32d_epi<T, l>(out, 2 * c - 1 + (lg >> 1), o0, v, sc, sh, pos0, Lout);
        } else {
          f32d_epi<T, l>(out, l < 4 ? c : 2 * c - 1 + ph, o0, acc[a] + acc2[a], sc, sh, pos0, Lout);
        }
      }
    }
  }
  // waves without a unit of this layer may have one of the next
  if (wave >= g::NU(l)) f32d_first<T, l + 1>(af, wn, wave, lane);
}

template <int T, int SRC, bool UPD>
__global__ __launch_bounds__(f32d::NTHR, 4) void dc_f32(ItemArgs args, DcIn p, DcF32P f, int ntile) {
  using namespace f32d;
  (void)args;
  if (!p.items) p.items = arg_items();
  using g = G<T>;
  __shared__ __attribute__((aligned(16))) float bufA[g::BUFA];
  __shared__ __attribute__((aligned(16))) float bufB[g::BUFB];
  __shared__ __attribute__((aligned(16))) float ksc[8][64], ksh[8][64], w8[64];
  const int W = p.Lin, tpw = (W + T - 1) / T;
  const int Gd = gridDim.x, j = blockIdx.x;
  const int t0 = (int)((int64_t)ntile * j / Gd), t1 = (int)((int64_t)ntile * (j + 1) / Gd);
  if (t0 >= t1) return;  // block-uniform
  for (int l = threadIdx.x >> 6; l < 8; l += NW) {
    const int o = threadIdx.x & 63, oc = o < C[l + 1] ? o : C[l + 1] - 1;
    ksc[l][o] = f.scale[l][oc];
    ksh[l][o] = f.shift[l][oc];
  }
  if (threadIdx.x < 56) w8[threadIdx.x] = f.wpk[8][threadIdx.x];
  const float s8 = f.scale[8][0], h8 = f.shift[8][0];
  float4 af[2] = {};
  for (int t = t0; t < t1; ++t) {
    const int b = t / tpw, u0 = (t - b * tpw) * T;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // keeps the layers' address arithmetic inside the loop
    f32d_stage<T, SRC, UPD>(bufA, p, b, u0 + LO[0], tid);
    f32d_first<T, 0>(af, f.wpk[0], __builtin_amdgcn_readfirstlane(tid >> 6), tid & 63);
    __syncthreads();
#define GW_LAYER(l, IN, OUT, DIV)                                                                                    \
  f32d_layer<T, l>(tid, IN, OUT, af, f.wpk[l], f.wpk[l + 1], ksc[l], ksh[l], u0 / (DIV) + LO[l + 1], W / (DIV));     \
  __syncthreads();
    GW_LAYER(0, bufA, bufB, 2)
    GW_LAYER(1, bufB, bufA, 4)
    GW_LAYER(2, bufA, bufB, 8)
    GW_LAYER(3, bufB, bufA, 16)
    GW_LAYER(4, bufA, bufB, 8)
    GW_LAYER(5, bufB, bufA, 4)
    GW_LAYER(6, bufA, bufB, 2)
    GW_LAYER(7, bufB, bufA, 1)
#undef GW_LAYER
    // output conv: one output a thread, 56 FMAs from LDS (an MFMA would use
    // one of its 16 rows)
    for (int c = tid; c < T; c += NTHR) {
      const int u = u0 + c;
      if (u >= W) break;
      const float4* row = reinterpret_cast<const float4*>(bufA + c * RS(8));
      const float4* wv = reinterpret_cast<const float4*>(w8);
      float acc = 0.0f;
#pragma unroll
      for (int k = 0; k < 7; ++k) {
        const float4 x0 = row[k * (RS(8) / 4)], x1 = row[k * (RS(8) / 4) + 1], w0 = wv[2 * k], w1 = wv[2 * k + 1];
        acc = fmaf(w0.x, x0.x, acc);
        acc = fmaf(w0.y, x0.y, acc);
        acc = fmaf(w0.z, x0.z, acc);
        acc = fmaf(w0.w, x0.w, acc);
        acc = fmaf(w1.x, x1.x, acc);
        acc = fmaf(w1.y, x1.y, acc);
        acc = fmaf(w1.z, x1.z, acc);
        acc = fmaf(w1.w, x1.w, acc);
      }
      const float v = fmaf(acc, s8, h8);
      if (p.noise) p.noise[(int64_t)b * W + u] = v;
      if (p.clean) {
        const Item& it = p.items[b];
        const int c0 = W - it.s - it.delay;
        if (u >= c0 && u < c0 + it.s) {
          const int64_t idx = it.out + (u - c0);
          p.clean[idx] = p.strain[idx] - v;
        }
      }
    }
    __syncthreads();  // bufA is the next tile's input
  }
}

template <int T, int SRC, bool UPD>
static hipError_t launch_dc_f32_t(const DcIn& p, const ItemArgs& args, const DcF32P& f, int n, int ncu,
                                  hipStream_t st) {
  const int64_t ntile = (int64_t)n * ((p.Lin + T - 1) / T);
  if (ntile > (int64_t)1 << 30) return hipErrorInvalidValue;
  static const int occ = [] {
    int k = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&k, dc_f32<T, SRC, UPD>, f32d::NTHR, 0) == hipSuccess && k > 0
               ? k
               : 1;
  }();
  const int64_t grid = std::min<int64_t>(ntile, (int64_t)occ * ncu);
  hipLaunchKernelGGL((dc_f32<T, SRC, UPD>), dim3((unsigned)grid), dim3(f32d::NTHR), 0, st, args, p, f, (int)ntile);
  return hipGetLastError();
}

template <int T>
static hipError_t launch_dc_f32_s(const DcIn& p, const ItemArgs& args, const DcF32P& f, int n, bool ring, int ncu,
                                  hipStream_t st) {
  if (!ring) return launch_dc_f32_t<T, SRC_DENSE, false>(p, args, f, n, ncu, st);
  return p.upd ? launch_dc_f32_t<T, SRC_RING, true>(p, args, f, n, ncu, st)
               : launch_dc_f32_t<T, SRC_RING, false>(p, args, f, n, ncu, st);
}

hipError_t launch_dc_f32(const DcIn& io, const ItemArgs& args, const float* const* wpk, const float* const* scale,
                         const float* const* shift, int n, bool ring, int cu_budget, hipStream_t st) {
  const int W = io.Lin;
  if (W < 16 || W % 16 || (io.upd && !ring)) return hipErrorInvalidValue;
  DcF32P f;
  for (int l = 0; l < 9; ++l) {
    f.wpk[l] = wpk[l];
    f.scale[l] = scale[l];
    f.shift[l] = shift[l];
  }
  DcIn q = io;
  if (!q.ldx) q.ldx = W;
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int ncu = cu_budget > 0 && cu_budget < cus ? cu_budget : cus;
  // Tile size.  A small tile spreads few windows over more CUs and ends its
  // chain of layers sooner; a large one wastes less on the halo (per output,
  // T = 128 computes 1.6 times what T = 512 does).  Two blocks share a CU.
  // Measured (us; one block on each CU, then per full round of two): T = 128
  // 17.5 and 23, 256: 21 and 31.5, 512: 30 and 50.  Windows of 21 x 32768:
  // n = 1: 17.7 (T = 256: 21.1); 2: 21.4 (25.3 at 128, 30.2 at 512); 4: 30.9
  // (33.4 at 256); 16: 101 (124 at 256, 178 at 128).
  auto cost = [&](int T, int one, int two) {
    const int64_t tiles = (int64_t)n * ((W + T - 1) / T);
    return tiles <= ncu ? (int64_t)one : (tiles + 2 * ncu - 1) / (2 * ncu) * two;
  };
  const int64_t c128 = cost(128, 175, 230), c256 = cost(256, 210, 315), c512 = cost(512, 300, 500);
  if (c128 <= c256 && c128 <= c512) return launch_dc_f32_s<128>(q, args, f, n, ring, ncu, st);
  if (c256 <= c512) return launch_dc_f32_s<256>(q, args, f, n, ring, ncu, st);
  return launch_dc_f32_s<512>(q, args, f, n, ring, ncu, st);
}

}  // namespace gw
