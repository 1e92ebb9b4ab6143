// Epilogue shared by the training convolutions (FP32 and split-BF16 matrix
// cores, whose accumulator fragments have the same layout).
#pragma once
#include "internal.h"

namespace gw {

typedef float tr_f32x4 __attribute__((ext_vector_type(4)));

// Training epilogue of one output channel o of a wave's columns: EPI_STATS
// writes z = acc + bias and sums (z, z^2); EPI_BNBWD turns the gradient of a
// into dh = acc (1 - a^2) and sums (dh, dh xhat).  FP64 sums over the lane's
// values, then over the 16 columns' lanes; out[0], out[1] get the wave's.
template <int MTB, int NPH, int NTW, int EPI>
__device__ __forceinline__ void train_out(const ConvP& p, const F32Train& tr,
                                               const tr_f32x4 (&acc)[NTW][NPH * MTB], double* out, int m, int r,
                                               int o, int b, int wcol0, int ncol, int lc) {
  double s0 = 0.0, s1 = 0.0;
  if (o < p.Co) {
    const int64_t row = ((int64_t)b * p.Co + o) * p.Lout;
    float mu = 0.f, is = 0.f, g = 0.f, be = p.bias ? p.bias[o] : 0.0f;
    if (EPI == EPI_BNBWD) {
      mu = tr.out.mean[o];
      is = tr.out.invstd[o];
      g = tr.out.gamma[o];
      be = tr.out.beta[o];
    }
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      const int col = wcol0 + 16 * t + lc;
      if (col >= ncol) continue;
      float v[NPH];
      if (EPI == EPI_STATS) {
#pragma unroll
        for (int ph = 0; ph < NPH; ++ph) {
          v[ph] = acc[t][ph * MTB + m][r] + be;
          s0 += (double)v[ph];
          s1 += (double)v[ph] * (double)v[ph];
        }
      } else {
        float zv[NPH];  // Lout = NPH ncol: every phase of the column is inside
        if (NPH == 2) {
          const float2 z2 = *reinterpret_cast<const float2*>(tr.z + row + 2 * col);
          zv[0] = z2.x;
          zv[NPH - 1] = z2.y;
        } else {
          zv[0] = tr.z[row + col];
        }
#pragma unroll
        for (int ph = 0; ph < NPH; ++ph) {
          const float xh = (zv[ph] - mu) * is, a = tanhf(fmaf(g, xh, be));
          v[ph] = acc[t][ph * MTB + m][r] * (1.0f - a * a);
          s0 += (double)v[ph];
          s1 += (double)v[ph] * (double)xh;
        }
      }
      if (NPH == 2)
        *reinterpret_cast<float2*>(p.y + row + 2 * col) = make_float2(v[0], v[NPH - 1]);
      else
        p.y[row + col] = v[0];
    }
  }
#pragma unroll
  for (int k = 1; k < 16; k <<= 1) {
    s0 += __shfl_xor(s0, k, 64);
    s1 += __shfl_xor(s1, k, 64);
  }
  if (lc == 0) {
    out[0] = s0;
    out[1] = s1;
  }
}

// The block's sums: the four waves' in order, to partial[o][blk][2].
template <int MTB>
__device__ __forceinline__ void train_sums(const double (&csum)[4][16 * MTB][2], double* partial, int o_lo, int Co,
                                           int nblk, int blk, int tid) {
  for (int e = tid; e < 32 * MTB; e += 256) {
    const int c = e >> 1, k = e & 1, o = o_lo + c;
    if (o < Co) partial[((int64_t)o * nblk + blk) * 2 + k] = ((csum[0][c][k] + csum[1][c][k]) + csum[2][c][k]) + csum[3][c][k];
  }
}

}  // namespace gw
