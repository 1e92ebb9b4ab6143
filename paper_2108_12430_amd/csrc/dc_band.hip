// Incremental DeepClean forward of the reference network: the noise ring of a
// stream's cache is brought up to date by computing only the outputs that
// changed, each from its receptive field.
//
// When a window has slid by a multiple of the total stride, an output keeps
// its value unless the newest samples or the window's left edge lie in its
// receptive field (93 samples on either side): outputs [0, zl) and [zr, W)
// change (cache_band in internal.h).  A block computes T of them through all
// nine layers with the activations in LDS, so only the noise ring has to be
// kept; outputs that did not change are copied from it by blocks of the same
// launch.  Tiles write changed outputs only and copies read the others, so no
// block depends on another.
//
// Arithmetic per output value: BF16 inputs (the snapshot's shadow), the
// model's BF16 weight fragments on v_mfma_f32_16x16x32_bf16 in K = tap x
// channel order, FP32 accumulation, folded normalisation and tanh in FP32,
// activations rounded to BF16.  An MFMA result depends on its own row and
// column only, so a value has the same bits whichever tile computes it, and
// an incremental update equals a full recompute.
//
// What bounds it: latency and the tanh's VALU issue (12.1k activations per
// 256 outputs); the matrix work is 344 MFMAs of 16 cycles a tile.  The kernel
// before kept every layer's activations as rings and walked a stream's dirty
// positions layer by layer in one block, about 21 dependent rounds.  Measured,
// 179 streams of 21 x 32768, strides 256, 512 and 1024 in turn: 125 -> 27 us a
// launch; all of 256: 83 -> 22 us; one stream: 78 -> 12 us.  (34, 26 and 14 us
// with the zones worked out by every wave and every stored row's address and
// range by every lane.)  T = 256: measured in that form, other sizes took 39
// (128), 37 (192) and 32 us (288) on the mixed strides, where 256 took 33, but
// 24, 24 and 27 us (256: 26) on strides of 256 and 12, 13 and 15 us (14) alone.
#include "internal.h"

namespace gw {
namespace band {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int T = 256;  // outputs per block
constexpr int NW = 8;
constexpr int NTHR = 64 * NW;
constexpr int C[10] = {21, 8, 16, 32, 64, 32, 16, 8, 8, 1};
constexpr int cip(int c) { return (c + 7) / 8 * 8; }
constexpr int rs(int c) { return (cip(c) / 8) % 2 ? cip(c) : cip(c) + 8; }  // an odd multiple of 16 bytes
constexpr int FRONT = 40;  // elements: a row of the widest transposed output, a multiple of 8
constexpr int LO[10] = {-93, -45, -21, -9, -3, -3, -3, -3, -3, 0};
constexpr int NR[10] = {T + 187, T / 2 + 91, T / 4 + 43, T / 8 + 19, T / 16 + 7,
                        T / 8 + 7, T / 4 + 7, T / 2 + 7, T + 6, T};
constexpr bool TR(int l) { return l >= 4 && l < 8; }
// columns: one per output row, or one input position of a transposed layer
// (column c makes rows 2c - 1 and 2c)
constexpr int NCOL(int l) {
  return l < 4 ? NR[l + 1] : l == 8 ? T : l == 4 ? T / 16 + 4 : l == 5 ? T / 8 + 4 : l == 6 ? T / 4 + 4 : T / 2 + 4;
}
constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }
constexpr int mx(int a, int b) { return a > b ? a : b; }
constexpr int NT(int l) { return cdiv(NCOL(l), 16); }
constexpr int KT(int l) { return TR(l) ? 4 : 7; }
constexpr int KS(int l) { return (KT(l) * cip(C[l]) + 31) / 32; }
constexpr int MT(int l) { return (C[l + 1] + 15) / 16; }
// both phases of a transposed layer with 8 output channels share a unit
constexpr bool BOTH(int l) { return l == 6 || l == 7; }
constexpr int QU(int l) { return BOTH(l) ? 1 : (TR(l) ? 2 : 1) * MT(l); }  // units per column group
constexpr int NP(int l) { return BOTH(l) ? 2 : 1; }                        // accumulators per column tile
constexpr int NTC(int l) { return cdiv(NT(l) * QU(l), NW); }
constexpr int NU(int l) { return cdiv(NT(l), NTC(l)) * QU(l); }
constexpr int NF(int l) { return NP(l) * KS(l); }  // weight fragments per unit
constexpr int FMAX = 8;
constexpr int SC(int l) { return l < 4 ? 2 : 1; }
// rows that columns read, or that the layer before stores (all of its column
// tiles': those past NR feed padded columns alone)
constexpr int ROWS(int l) {
  return mx(mx(SC(l) * (16 * NT(l) - 1) + KT(l), NR[l]), l > 0 ? (TR(l - 1) ? 32 : 16) * NT(l - 1) : 0);
}
constexpr int HALF(int l) { return l < 4 ? (ROWS(l) + 1) / 2 : 0; }  // even rows, then odd rows
constexpr int prow(int l, int r) { return l < 4 ? (r & 1) * HALF(l) + (r >> 1) : r; }
constexpr int SZ(int l) { return (HALF(l) ? 2 * HALF(l) : ROWS(l)) * rs(C[l]); }
constexpr int BUFA = mx(mx(mx(SZ(0), SZ(2)), mx(SZ(4), SZ(6))), SZ(8));
constexpr int BUFB = mx(mx(SZ(1), SZ(3)), mx(SZ(5), SZ(7)));
constexpr bool fit(int l) { return l == 9 || (NF(l) <= FMAX && NU(l) <= NW && fit(l + 1)); }
static_assert(fit(0), "one round of units of at most FMAX fragments per layer");
static_assert(ROWS(0) <= NTHR, "one input row per thread");

struct P {
  const uint16_t* wpk[9];
  const float* scale[9];
  const float* shift[9];
  const float* strain;
  float* noise;
  float* clean;
  size_t ring;  // byte offset of the noise ring in a cache
  int W, tiles, copies;  // an item's blocks: tiles, then copies
};

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){lo, hi}, b2));
}

// all of wave `wave`'s weight fragments of layer l
template <int l>
__device__ __forceinline__ void frags(uint4 (&wf)[FMAX], const uint16_t* w, int wave, int lane) {
  if constexpr (l < 9) {
    if (wave >= NU(l)) return;  // wave-uniform
    const uint4* q = reinterpret_cast<const uint4*>(w) + (wave % QU(l)) * NF(l) * 64 + lane;
#pragma unroll
    for (int i = 0; i < NF(l); ++i) wf[i] = q[i * 64];
  }
}

// normalisation + tanh of four channels of an output row; zeros outside the
// signal (the next layer's padding).  Rows are not masked: row -1 of a
// transposed layer lands in the pad before the buffer.
__device__ __forceinline__ void epi(uint16_t* dst, f32x4 v, const float4& sc, const float4& sh, bool live) {
  const uint2 d = make_uint2(pack2(tanhf(fmaf(v[0], sc.x, sh.x)), tanhf(fmaf(v[1], sc.y, sh.y))),
                             pack2(tanhf(fmaf(v[2], sc.z, sh.z)), tanhf(fmaf(v[3], sc.w, sh.w))));
  *reinterpret_cast<uint2*>(dst) = live ? d : make_uint2(0u, 0u);
}

__device__ __forceinline__ float swap32(float a, float b) {  // lanes 0..31: a's; 32..63: b's lanes 0..31
  return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false)[0]);
}

template <int l, typename OutFn>
__device__ __forceinline__ void layer(int tid, const uint16_t* in, uint16_t* out, uint4 (&wf)[FMAX],
                                      const uint16_t* wn, const float* ksc, const float* ksh, int pos0, int Lout,
                                      OutFn final_out) {
  constexpr int CIP = cip(C[l]), RSI = rs(C[l]), NTn = NT(l), NTCl = NTC(l), NPl = NP(l), KSn = KS(l);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & 15, lg = lane >> 4;
  if (wave >= NU(l)) {  // wave-uniform
    frags<l + 1>(wf, wn, wave, lane);
    return;
  }
  const int q = wave % QU(l), nt0 = wave / QU(l) * NTCl;
  const int ph = q / MT(l), mt = q % MT(l);
  const uint16_t* colbase = in + (nt0 * 16 + lc) * RSI;
  f32x4 acc[NTCl][NPl];
#pragma unroll
  for (int a = 0; a < NTCl; ++a)
#pragma unroll
    for (int k = 0; k < NPl; ++k) acc[a][k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KSn; ++ks) {
    const int kappa = 32 * ks + 8 * lg, j0 = kappa / CIP, i0 = kappa - j0 * CIP;
    const int jj = j0 < KT(l) ? j0 : KT(l) - 1;  // K padding: zero weights, a row of finite values
    const int row = l < 4 ? (jj & 1) * HALF(l) + (jj >> 1) : jj;
    uint4 bv[NTCl];
#pragma unroll
    for (int a = 0; a < NTCl; ++a) {
      const int aa = a < NTn - nt0 ? a : NTn - 1 - nt0;  // past the last tile: that one again, not stored
      bv[a] = *reinterpret_cast<const uint4*>(colbase + (row + 16 * aa) * RSI + i0);
    }
#pragma unroll
    for (int a = 0; a < NTCl; ++a)
#pragma unroll
      for (int k = 0; k < NPl; ++k)
        acc[a][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[k * KSn + ks]),
                                                            __builtin_bit_cast(bf16x8, bv[a]), acc[a][k], 0, 0, 0);
  }
  frags<l + 1>(wf, wn, wave, lane);
  // lane (lc, lg) holds rows 4 lg .. 4 lg + 3 of column 16 (nt0 + a) + lc; a
  // tile's rows start TSTEP elements after those of the tile before
  constexpr int RSO = l < 8 ? rs(C[l + 1]) : 0, RPT = TR(l) ? 32 : 16, TSTEP = (l + 1 < 4 ? RPT / 2 : RPT) * RSO;
  if constexpr (l == 8) {
    if (lg == 0)
#pragma unroll
      for (int a = 0; a < NTCl; ++a)
        if (nt0 + a < NTn) final_out((nt0 + a) * 16 + lc, fmaf(acc[a][0][0], ksc[0], ksh[0]));
  } else if constexpr (C[l + 1] == 8) {
    // eight channels fill lanes 0..31: the upper lanes take the other phase,
    // or the next column tile
    const int o0 = 4 * (lg & 1);
    const float4 sc = *reinterpret_cast<const float4*>(ksc + o0), sh = *reinterpret_cast<const float4*>(ksh + o0);
    constexpr int ST = NPl == 2 ? 1 : 2;
    const int r0 = NPl == 2 ? 2 * lc - 1 + (lg >> 1) : 16 * (lg >> 1) + lc;  // row of tile 0
    uint16_t* dst = out + prow(l + 1, r0) * RSO + o0 + nt0 * TSTEP;
    const int u0 = pos0 + RPT * nt0 + r0;
#pragma unroll
    for (int a = 0; a < NTCl; a += ST) {
      if (nt0 + a >= NTn) break;
      f32x4 v;
      const bool pair = NPl == 2 || (a + 1 < NTCl && nt0 + a + 1 < NTn);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        v[r] = swap32(acc[a][0][r], NPl == 2 ? acc[a][NPl - 1][r] : acc[a + 1 < NTCl ? a + 1 : a][0][r]);
      if (!pair && lg >= 2) continue;
      epi(dst + a * TSTEP, v, sc, sh, u0 + RPT * a >= 0 && u0 + RPT * a < Lout);
    }
  } else {
    const int o0 = 16 * mt + 4 * lg;
    const float4 sc = *reinterpret_cast<const float4*>(ksc + o0), sh = *reinterpret_cast<const float4*>(ksh + o0);
    const int r0 = TR(l) ? 2 * lc - 1 + ph : lc;
    uint16_t* dst = out + prow(l + 1, r0) * RSO + o0 + nt0 * TSTEP;
    const int u0 = pos0 + RPT * nt0 + r0;
#pragma unroll
    for (int a = 0; a < NTCl; ++a) {
      if (nt0 + a >= NTn) break;
      epi(dst + a * TSTEP, acc[a][0], sc, sh, u0 + RPT * a >= 0 && u0 + RPT * a < Lout);
    }
  }
}

// first output of the right zone's tiles
__host__ __device__ constexpr int right0(int zr) { return zr & ~15; }

}  // namespace band

// the outputs that change when a window of W samples slides by shift
void cache_band_zones(int shift, int W, int* zl, int* zr) {
  using namespace band;
  CacheGeo g[9];
  int L = W;
  for (int l = 0; l < 9; ++l) {
    const int Lo = l < 4 ? L / 2 : l < 8 ? 2 * L : L;
    g[l] = CacheGeo{TR(l) ? 1 : 0, C[l], C[l + 1], 7, l == 8 ? 1 : 2, 3, TR(l) ? 1 : 0, L, Lo, W / Lo, l < 8, l == 8};
    L = Lo;
  }
  cache_band(g, 8, shift, W, zl, zr);
}

int cache_band_tiles(int zl, int zr, int W) {
  return band::cdiv(zl, band::T) + band::cdiv(W - band::right0(zr), band::T);
}

__global__ __launch_bounds__(band::NTHR, 4) void cache_band_kernel(const CacheItem* items, const void* arena,
                                                                    band::P p) {
  using namespace band;
  __shared__ __attribute__((aligned(16))) uint16_t padA[FRONT + BUFA];
  __shared__ __attribute__((aligned(16))) uint16_t padB[FRONT + BUFB];
  uint16_t *const bufA = padA + FRONT, *const bufB = padB + FRONT;
  __shared__ __attribute__((aligned(16))) float ksc[9][64], ksh[9][64];
  const int per = p.tiles + p.copies, item = (int)blockIdx.x / per, t = (int)blockIdx.x - item * per;
  const CacheItem it = items[item];
  const int W = p.W, tid0 = threadIdx.x;
  const int zl = it.zl, zr = it.zr;
  float* ring = reinterpret_cast<float*>(reinterpret_cast<char*>(it.cache) + p.ring);
  const int s0 = W - it.s - it.delay;  // clean span [s0, s0 + s)
  auto emit = [&](int k, float v) {
    if (p.noise) p.noise[(int64_t)item * W + k] = v;
    if (p.clean && k >= s0 && k < s0 + it.s) p.clean[it.out + (k - s0)] = p.strain[it.out + (k - s0)] - v;
  };
  if (t >= p.tiles) {
    // copies of the outputs that did not change, 8 a thread
    const int k0 = p.noise ? 0 : s0, k1 = p.noise ? W : s0 + it.s;
    const int base = k0 + (t - p.tiles) * 8 * NTHR;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = base + j * NTHR + tid0;
      if (k >= k1 || k < zl || k >= zr) continue;
      int sl = it.T + k;
      if (sl >= W) sl -= W;
      emit(k, ring[sl]);
    }
    return;
  }
  const int ntl = (zl + T - 1) / T;
  const int u0 = t < ntl ? t * T : right0(zr) + (t - ntl) * T;
  if (u0 >= W) return;  // block-uniform: this item has fewer tiles
  const int w0 = t < ntl ? 0 : zr, w1 = t < ntl ? zl : W;  // outputs this tile may write
  {
    // input row r: sample u0 - 93 + r of every channel, one row a thread
    const int r = tid0, q = u0 + LO[0] + r;
    const bool live = q >= 0 && q < W;
    const uint16_t* sh = reinterpret_cast<const uint16_t*>(arena) + it.shadow;
    int at = it.in_head + (live ? q : 0);
    if (at >= W) at -= W;
    uint32_t v[24];
#pragma unroll
    for (int i = 0; i < 24; ++i) v[i] = i < C[0] ? sh[(int64_t)(i < C[0] ? i : 0) * W + at] : 0u;
    if (r < ROWS(0)) {
      uint4* d = reinterpret_cast<uint4*>(bufA + prow(0, r) * rs(C[0]));
#pragma unroll
      for (int k = 0; k < 3; ++k)
        d[k] = live ? make_uint4(v[8 * k] | v[8 * k + 1] << 16, v[8 * k + 2] | v[8 * k + 3] << 16,
                                 v[8 * k + 4] | v[8 * k + 5] << 16, v[8 * k + 6] | v[8 * k + 7] << 16)
                    : make_uint4(0u, 0u, 0u, 0u);
    }
  }
  for (int l = tid0 >> 6; l < 9; l += NW) {
    const int o = tid0 & 63, oc = o < C[l + 1] ? o : C[l + 1] - 1;
    ksc[l][o] = p.scale[l][oc];
    ksh[l][o] = p.shift[l][oc];
  }
  uint4 wf[FMAX];
  frags<0>(wf, p.wpk[0], __builtin_amdgcn_readfirstlane(tid0 >> 6), tid0 & 63);
  __syncthreads();
  auto fin = [&](int c, float v) {
    const int k = u0 + c;
    if (k < w0 || k >= w1) return;
    int sl = it.T + k;
    if (sl >= W) sl -= W;
    ring[sl] = v;
    emit(k, v);
  };
#define GW_LAYER(l, IN, OUT, DIV)                                                                                    \
  layer<l>(tid0, IN, OUT, wf, p.wpk[(l + 1) % 9], ksc[l], ksh[l], u0 / (DIV) + LO[l + 1], W / (DIV), fin);           \
  if (l < 8) __syncthreads();
  GW_LAYER(0, bufA, bufB, 2)
  GW_LAYER(1, bufB, bufA, 4)
  GW_LAYER(2, bufA, bufB, 8)
  GW_LAYER(3, bufB, bufA, 16)
  GW_LAYER(4, bufA, bufB, 8)
  GW_LAYER(5, bufB, bufA, 4)
  GW_LAYER(6, bufA, bufB, 2)
  GW_LAYER(7, bufB, bufA, 1)
  GW_LAYER(8, bufA, bufB, 1)
#undef GW_LAYER
}

// tiles: the most cache_band_tiles of the items; smax: the longest clean span
hipError_t launch_cache_band(const CacheItem* items, int n, const void* arena, const CacheLayerP& P, int tiles, int smax,
                             const float* strain, float* noise, float* clean, hipStream_t st) {
  using namespace band;
  if (n < 1 || P.L != 9 || P.W % 16) return hipErrorInvalidValue;
  band::P p{};
  for (int l = 0; l < 9; ++l) {
    p.wpk[l] = P.wpk[l];
    p.scale[l] = P.scale[l];
    p.shift[l] = P.shift[l];
  }
  p.strain = strain;
  p.noise = noise;
  p.clean = clean;
  p.ring = P.off[8];
  p.W = P.W;
  p.tiles = tiles;
  p.copies = noise ? cdiv(P.W, 8 * NTHR) : clean ? cdiv(smax, 8 * NTHR) : 0;
  const int64_t blocks = (int64_t)n * (tiles + p.copies);
  if (blocks < 1) return hipSuccess;
  if (blocks > ((int64_t)1 << 31) - 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(cache_band_kernel, dim3((unsigned)blocks), dim3(NTHR), 0, st, items, arena, p);
  return hipGetLastError();
}

}  // namespace gw
