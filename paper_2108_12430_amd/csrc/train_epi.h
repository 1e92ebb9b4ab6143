// Epilogue shared by the training convolutions (FP32 and split-BF16 matrix
// cores, whose accumulator fragments have the same layout): lane (lc, lg) of a
// wave holds channels 16 m + 4 lg + r of columns 16 (wave NTW + t) + lc, and of
// both phases of a transposed layer.
#pragma once
#include "internal.h"

namespace gw {

typedef float tr_f32x4 __attribute__((ext_vector_type(4)));

// floats of LDS it needs: the block's outputs, [channel][position]
constexpr int train_tile_floats(int co, int tno) { return co * (tno + 4); }

// EPI_STATS writes z = acc + bias and sums (z, z^2); EPI_BNBWD turns the
// gradient of a into dh = acc (1 - a^2) and sums (dh, dh xhat).  The
// accumulators go through LDS so that every lane then works on four
// consecutive positions of one channel: whole 16-byte loads and stores, no
// idle lanes in the layers of eight channels, and 256 / C_out threads per
// channel, within one wave, whose FP64 sums need a few lane exchanges and no
// barrier.  (Done from the fragments, a layer of eight channels left half the
// lanes idle through the tanh and took 64 exchanges per wave: the eight adjoint
// convolutions of a batch-32 step took 300 us, 255 here.)  Sums are added in a
// fixed order.  C_out is 8, 16, 32 or 64; ot may alias what the
// MFMAs read: the caller's waves meet here first.
template <int MTB, int NPH, int NTW, int EPI>
__device__ __forceinline__ void train_epilogue(const ConvP& p, const F32Train& tr,
                                               const tr_f32x4 (&acc)[NTW][NPH * MTB], float* ot, int b, int col0,
                                               int blk, int nblk, int tid) {
  constexpr int TNO = 64 * NTW * NPH, OS = TNO + 4;
  const int lane = tid & 63, wave = tid >> 6, lc = lane & 15, lg = lane >> 4;
  const int Co = p.Co, tpc = 256 / Co, sh = __builtin_ctz(tpc);  // threads per channel
  const int o = tid >> sh, k = tid & (tpc - 1);
  const int64_t row = ((int64_t)b * Co + o) * p.Lout;
  const int u0 = NPH * col0 + 4 * k, us = 4 * tpc, ue = min(NPH * col0 + TNO, p.Lout);
  const bool vec = ((p.Lout & 3) | (reinterpret_cast<uintptr_t>(p.y) & 15) |
                    (EPI == EPI_BNBWD ? reinterpret_cast<uintptr_t>(tr.z) & 15 : 0)) == 0;
  __syncthreads();
#pragma unroll
  for (int m = 0; m < MTB; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ol = 16 * m + 4 * lg + r;
      if (ol >= Co) continue;
      float* d = ot + ol * OS;
#pragma unroll
      for (int t = 0; t < NTW; ++t) {
        const int c = (wave * NTW + t) * 16 + lc;
        if (NPH == 2)
          *reinterpret_cast<float2*>(d + 2 * c) = make_float2(acc[t][m][r], acc[t][(NPH - 1) * MTB + m][r]);
        else
          d[c] = acc[t][m][r];
      }
    }
  float c0 = p.bias ? p.bias[o] : 0.0f, mu = 0.f, is = 0.f, g = 0.f, be = 0.f;
  if (EPI == EPI_BNBWD) {
    mu = tr.out.mean[o];
    is = tr.out.invstd[o];
    g = tr.out.gamma[o];
    be = tr.out.beta[o];
  }
  __syncthreads();
  const float* src = ot + o * OS + 4 * k;
  double s0 = 0.0, s1 = 0.0;
  constexpr int B = EPI == EPI_BNBWD ? 4 : 1;  // z loads in flight
  for (int u = u0, i = 0; u < ue; u += B * us, i += B * us) {
    float4 zv[B];
    if (EPI == EPI_BNBWD) {
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const int v = u + j * us;
        zv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (vec && v + 4 <= ue) {
          zv[j] = *reinterpret_cast<const float4*>(tr.z + row + v);
        } else {
          float* d = &zv[j].x;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (v + e < ue) d[e] = tr.z[row + v + e];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int v = u + j * us;
      if (v >= ue) break;
      const int live = ue - v;  // positions of the four that exist
      float4 y = *reinterpret_cast<const float4*>(src + i + j * us);
      float* yd = &y.x;
      const float* zd = &zv[j].x;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (EPI == EPI_STATS) {
          yd[e] += c0;
          if (e < live) {
            s0 += (double)yd[e];
            s1 += (double)yd[e] * (double)yd[e];
          }
        } else {
          const float xh = (zd[e] - mu) * is, a = tanhf(fmaf(g, xh, be));
          yd[e] *= 1.0f - a * a;
          if (e < live) {
            s0 += (double)yd[e];
            s1 += (double)yd[e] * (double)xh;
          }
        }
      }
      float* out = p.y + row + v;
      if (vec && live >= 4) {
        *reinterpret_cast<float4*>(out) = y;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < live) out[e] = yd[e];
      }
    }
  }
  for (int d = 1; d < tpc; d <<= 1) {
    s0 += __shfl_xor(s0, d, 64);
    s1 += __shfl_xor(s1, d, 64);
  }
  if (k == 0) {
    double* out = tr.partial + ((int64_t)o * nblk + blk) * 2;
    out[0] = s0;
    out[1] = s1;
  }
}

// what train_epilogue takes
inline bool train_epilogue_fits(int Co, int mtb) { return Co == 16 * mtb ? (Co & (Co - 1)) == 0 && Co <= 64 : mtb == 1 && Co == 8; }

}  // namespace gw
