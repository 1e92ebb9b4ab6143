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
// One launch runs every layer, so that no layer pays for a launch of its own to
// fill and drain.  Its 1536 blocks are three for each place on the chip (two per
// CU), shared out among the layers.  A block's sums are FP32, so a layer has so
// many blocks that no sum takes more products than in the per-layer launches of
// 256 blocks (wgrad_partial): 256 chains, a chain being one K slice of a block,
// or 512 where those split their chunks in two.  (512 blocks, all resident and
// ending together, left chains up to 4.4 times as long.)  No wave holds more than
// ten accumulator tiles: 128 registers, so that two blocks of eight waves share a
// CU, hold them and a chunk's loads without spilling.
//
// Measured, batch 32 x 21 x 32768: nine launches with operands read from memory
// as they are and a launch pair per layer for the reduction 384 us (and 190 us
// more to write dz and the activations); nine launches of this kernel's
// blocks, with the reduction, the output conv's bias sum and the zero fill
// 314 us; one launch and its reduction 207 us (512 blocks: 198; at batch 128 712
// and 745; matrix cores 70 us, memory at copy rate 106 us).  512 blocks that close
// their sums one to five times on the way: 248 us, the chunks' loop is slower with
// the closing in it.
#include "internal.h"

namespace gw {
namespace wg2 {

typedef float f32x4 __attribute__((ext_vector_type(4)));

enum Mode : int { RAW = 0, ACT = 1, DZ = 2 };

// CA rows, CC columns' channels, stride, chunk of times, the operands' modes
template <int CA_, int CC_, int S_, int WT_, int PM_, int QM_>
struct Cfg {
  static constexpr int CA = CA_, CC = CC_, S = S_, WT = WT_, NW = 8, PM = PM_, QM = QM_;
  static constexpr int NTHR = 64 * NW;
  static constexpr int NK = CC * 7, MA = (CA + 15) / 16, NB = (NK + 15) / 16;
  static constexpr int KC = WT / 16;                    // K steps per chunk
  static constexpr int NT = MA * NB;                    // accumulator tiles: at most ten a wave
  static constexpr int NS = NT > 40 ? 1 : NT > 20 ? 2 : NT > 10 ? 4 : KC < NW ? KC : NW;  // K slices
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
  // The output conv has one row and eight channels: the products are the same
  // with the operands exchanged and the taps in reverse, and fill 8 x 7 of one
  // tile instead of 1 x 56 of four.
  static constexpr bool REV = CC == 1;
  static_assert(!REV || QW / 4 <= NTHR, "one item of Q per thread");
  static_assert(WT % 16 == 0 && KC % NS == 0 && NW % NS == 0 && (NS & (NS - 1)) == 0, "slices");
};

struct Opnd {
  const float* x;
  BnBwdP bn;
};

struct P2 {
  Opnd p, q;
  int Lp, Lq, tchunks, nchunk, blocks;
  float* partial;  // [blocks][CA * NK]
  double* bsum;    // [blocks] sums of Q (REV)
};

struct All {
  P2 e[9];
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

// block bi of layer p
template <class K>
__device__ __forceinline__ void wgrad2_body(const wg2::P2& p, int bi, float* lds, float* cp, float* cq) {
  using namespace wg2;
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
  int bp[K::NBW];
#pragma unroll
  for (int u = 0; u < K::NBW; ++u) {
    const int n0 = 16 * (grp * K::NBW + u) + lr, nn = n0 < K::NK ? n0 : K::NK - 1, c = nn / 7, j = nn - 7 * c;
    bp[u] = (K::S == 2 ? (2 * c + ((1 + j) & 1)) * K::QP + (1 + j) / 2 : c * K::QP + 1 + j) + 4 * lk;
  }
  f32x4 acc[K::MA][K::NBW];
#pragma unroll
  for (int m = 0; m < K::MA; ++m)
#pragma unroll
    for (int u = 0; u < K::NBW; ++u) acc[m][u] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int G = p.blocks;
  const int c0 = (int)((int64_t)p.nchunk * bi / G), c1 = (int)((int64_t)p.nchunk * (bi + 1) / G);
  double bsum = 0.0;  // REV: this thread's share of the sum of Q
  if (c0 < c1) fetch(c0);
  for (int chunk = c0; chunk < c1; ++chunk) {
    __syncthreads();  // the constants are there; the previous chunk's reads are done
    stage(chunk);
    if (K::REV && tid >= 1 && tid <= PC)  // the chunk's own times, without the taps' reach
      bsum += ((double)qv[0].x + (double)qv[0].y) + ((double)qv[0].z + (double)qv[0].w);
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
        for (int e = 0; e < 4; ++e) bv[e] = Qs[bp[u] + 16 * ks + e];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int m = 0; m < K::MA; ++m)
            acc[m][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&av[m])[e], bv[e],
                                                             acc[m][u], 0, 0, 0);
      }
    }
  }
  if (K::REV) {
    __syncthreads();
    for (int off = 32; off > 0; off >>= 1) bsum += __shfl_down(bsum, off, 64);
    double* bs = reinterpret_cast<double*>(lds);
    if (lane == 0) bs[wave] = bsum;
    __syncthreads();
    if (tid == 0) {
      double t = bs[0];
      for (int w = 1; w < K::NW; ++w) t += bs[w];
      p.bsum[bi] = t;
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
  float* out = p.partial + (int64_t)bi * (K::CA * K::NK);
#pragma unroll
  for (int m = 0; m < K::MA; ++m)
#pragma unroll
    for (int u = 0; u < K::NBW; ++u) {
      const int nn = 16 * (grp * K::NBW + u) + lr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * m + 4 * lk + r;
        if (a < K::CA && nn < K::NK) out[a * K::NK + (K::REV ? K::NK - 1 - nn : nn)] = acc[m][u][r];
      }
    }
}

namespace wg2 {
typedef Cfg<8, 21, 2, 128, DZ, RAW> C0;
typedef Cfg<16, 8, 2, 256, DZ, ACT> C1;
typedef Cfg<32, 16, 2, 128, DZ, ACT> C2;
typedef Cfg<64, 32, 2, 64, DZ, ACT> C3;
typedef Cfg<64, 32, 2, 64, ACT, DZ> C4;
typedef Cfg<32, 16, 2, 128, ACT, DZ> C5;
typedef Cfg<16, 8, 2, 256, ACT, DZ> C6;
typedef Cfg<8, 8, 2, 256, ACT, DZ> C7;
typedef Cfg<8, 1, 1, 512, ACT, RAW> C8;

// each layer's blocks.  chains_ok holds from 32, 64, 64, 256, 256 and then 64 on;
// with 124 for layer 0 and those the launch takes 222 us, as long blocks end alone
constexpr int kShare[9] = {256, 128, 128, 256, 256, 128, 128, 128, 128};

constexpr int mx(int a, int b) { return a > b ? a : b; }
constexpr int LDS =
    mx(mx(mx(mx(C0::LDS, C1::LDS), mx(C2::LDS, C3::LDS)), mx(mx(C4::LDS, C5::LDS), mx(C6::LDS, C7::LDS))), C8::LDS);
static_assert(LDS * 4 + 12 * 64 * 4 <= 80 * 1024, "two blocks per CU");

struct Geo2 {
  int wt, ca, nk, ns;
};
template <class K>
constexpr Geo2 geo() {
  return {K::WT, K::CA, K::NK, K::NS};
}
constexpr Geo2 kGeo[9] = {geo<C0>(), geo<C1>(), geo<C2>(), geo<C3>(), geo<C4>(), geo<C5>(), geo<C6>(), geo<C7>(), geo<C8>()};

// layer l's chains at least those of its per-layer launch
constexpr bool chains_ok(int l) {
  return l == 9 || (kShare[l] * kGeo[l].ns >= (l == 1 || l >= 6 ? 512 : 256) && chains_ok(l + 1));
}
static_assert(chains_ok(0), "weight gradients: FP32 sums of too many products");

int64_t chunks(int l, int n, int Lp) { return (int64_t)n * ((Lp + kGeo[l].wt - 1) / kGeo[l].wt); }
int blocks(int l, int n, int Lp) { return (int)std::min<int64_t>(chunks(l, n, Lp), kShare[l]); }
}  // namespace wg2

__global__ __launch_bounds__(512, 4) void wgrad2(wg2::All t) {
  using namespace wg2;
  __shared__ __attribute__((aligned(16))) float lds[wg2::LDS];
  __shared__ float cp[6 * 64], cq[6 * 64];
  int bi = blockIdx.x, s = 0;
  while (bi >= t.e[s].blocks) bi -= t.e[s++].blocks;  // block-uniform
#define GW_SUB(i, K) \
  case i: wgrad2_body<K>(t.e[i], bi, lds, cp, cq); break;
  switch (s) {
    GW_SUB(0, C0)
    GW_SUB(1, C1)
    GW_SUB(2, C2)
    GW_SUB(3, C3)
    GW_SUB(4, C4)
    GW_SUB(5, C5)
    GW_SUB(6, C6)
    GW_SUB(7, C7)
    GW_SUB(8, C8)
  }
#undef GW_SUB
}

// Sums of the partials, one launch: a block takes 64 weights of one layer, its four waves a quarter of the partials each (in order), FP64.
// The last block adds the output conv's bias sums and clears the gradients
// that are exactly zero: the biases under batch normalisation and the running
// statistics.
struct Wg2Red {
  const float* partial;
  float* dw;
  int nw, G, blocks;
};
struct Wg2Zero {
  float* p;
  int n;
};
struct Wg2RedTab {
  Wg2Red e[9];
  const double* bsum;
  float* db;
  int nb;
  Wg2Zero zero[16];
};
__global__ __launch_bounds__(256) void wgrad2_reduce(Wg2RedTab t) {
  __shared__ double s[4][64];
  int blk = blockIdx.x, l = 0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (blk == (int)gridDim.x - 1) {
    for (int z = 0; z < 16; ++z)
      for (int i = threadIdx.x; i < t.zero[z].n; i += 256) t.zero[z].p[i] = 0.0f;
    if (threadIdx.x == 0) {
      double acc = 0.0;
      for (int g = 0; g < t.nb; ++g) acc += t.bsum[g];
      *t.db = (float)acc;
    }
    return;
  }
  while (blk >= t.e[l].blocks) blk -= t.e[l++].blocks;
  const Wg2Red& q = t.e[l];
  const int e = blk * 64 + lane;
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

static size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Lp: per layer, the length of its P (the conv's output, the transposed
// conv's input)
size_t wgrad2_scratch_bytes(int n, const int* Lp) {
  size_t b = 0;
  for (int l = 0; l < 9; ++l) b += up256(4 * (size_t)wg2::blocks(l, n, Lp[l]) * wg2::kGeo[l].ca * wg2::kGeo[l].nk);
  return b + up256(8 * (size_t)wg2::blocks(8, n, Lp[8]));
}

hipError_t launch_wgrad2(const Wg2Args (&a)[9], void* scratch, float* dbias, const F32Range* zero, int nzero,
                         hipStream_t st) {
  using namespace wg2;
  All t{};
  Wg2RedTab r{};
  if (nzero > 16) return hipErrorInvalidValue;
  char* at = reinterpret_cast<char*>(scratch);
  int grid = 0, rgrid = 1;
  for (int l = 0; l < 9; ++l) {
    const Wg2Args& w = a[l];
    const Geo2& g = kGeo[l];
    const int64_t nch = chunks(l, w.n, w.Lp);
    if (nch > (int64_t)1 << 30) return hipErrorInvalidValue;
    P2& p = t.e[l];
    p.p = {w.p, w.pbn};
    p.q = {w.q, w.qbn};
    p.Lp = w.Lp;
    p.Lq = w.Lq;
    p.tchunks = (w.Lp + g.wt - 1) / g.wt;
    p.nchunk = (int)nch;
    p.blocks = blocks(l, w.n, w.Lp);
    p.partial = reinterpret_cast<float*>(at);
    const int nw = g.ca * g.nk;
    at += up256(4 * (size_t)p.blocks * nw);
    grid += p.blocks;
    r.e[l] = {p.partial, w.dw, nw, p.blocks, (nw + 63) / 64};
    rgrid += r.e[l].blocks;
  }
  t.e[8].bsum = reinterpret_cast<double*>(at);
  r.bsum = t.e[8].bsum;
  r.db = dbias;
  r.nb = t.e[8].blocks;
  for (int z = 0; z < nzero; ++z) r.zero[z] = {zero[z].p, zero[z].n};
  hipLaunchKernelGGL(wgrad2, dim3(grid), dim3(512), 0, st, t);
  hipLaunchKernelGGL(wgrad2_reduce, dim3(rgrid), dim3(256), 0, st, r);
  return hipGetLastError();
}

}  // namespace gw
