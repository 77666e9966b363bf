// Backward pass of the networks' convolutions (training).
//
// The gradients are those of the im2col products: every product runs on
// v_mfma_f32_32x32x16_bf16 over the same groups of 16 depth values in the same
// order, and every FP32 sum outside it keeps its order, so weights, biases
// and input gradients have the bits of im2col + product + col2im. What is
// gone is the matrices themselves (9 values in HBM for every activation, as
// BF16 for the weight gradient and as FP32 for the input gradient).
#include <algorithm>
#include <cstdint>

#include "nn_internal.h"

namespace seg {
namespace nn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// two floats rounded to BF16 (nearest even), the first in the low half
__device__ __forceinline__ uint32_t pk(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}

// ---------------------------------------------------- mask and bias gradient
// One pass over a layer's output gradient dY [C][N]: the ReLU mask (MODE
// MASK: dY = 0 where not Y > 0), or the gradient itself from the output layer
// (MODE OUTER: dY[c][n] = wo[c] gl[n], the 1 x 1 layer's BF16 product of depth
// one, masked), and the bias gradient. That is the sum of 256 strided chains
// per channel (chain t: n = t, t + 256, ...), each in order, then a tree over
// the chains (k_grad_reduce). A block takes 32 chains of one channel: all its
// threads load, through LDS, and 32 of them add, so the chains' length does
// not hold the loads back. The thirteen layers of the summary network's step
// of 32 patches of 64 x 64 take 112 us, mask included, where a mask pass and
// one block per channel with a load per add took 1,084 us.
enum { BIAS_ONLY = 0, BIAS_MASK = 1, BIAS_OUTER = 2 };
constexpr int BG_ROWS = 64;   // chain elements per step

template <int MODE>
__global__ __launch_bounds__(256) void k_bias_mask(float* __restrict__ dY, const float* __restrict__ Y,
                                                   const float* __restrict__ gl, const uint16_t* __restrict__ wo,
                                                   float* __restrict__ part, long long N) {
  __shared__ float sh[BG_ROWS][33];
  const int c = blockIdx.x, tid = threadIdx.x, l = tid & 31, r = tid >> 5;
  const int chain = blockIdx.y * 32 + l;
  float* dy = dY + (long long)c * N;
  const float* y = MODE == BIAS_ONLY ? nullptr : Y + (long long)c * N;
  float w = 0.f;
  if constexpr (MODE == BIAS_OUTER) w = __uint_as_float((uint32_t)wo[c] << 16);
  const long long rows = (N + 255) / 256;
  const long long mine = N > chain ? (N - chain + 255) / 256 : 0;   // elements of this lane's chain
  float v[8], m[8];
  auto load = [&](long long k0) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long long n = min((k0 + u * 8 + r) * 256 + chain, N - 1);
      v[u] = MODE == BIAS_OUTER ? gl[n] : dy[n];
      if constexpr (MODE != BIAS_ONLY) m[u] = y[n];
    }
  };
  float s = 0.f;
  load(0);
  for (long long k0 = 0; k0 < rows; k0 += BG_ROWS) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long long n = (k0 + u * 8 + r) * 256 + chain;
      float x = v[u];
      if constexpr (MODE == BIAS_OUTER) x = w * __uint_as_float(pk(x, 0.f) << 16) + 0.f;
      if constexpr (MODE != BIAS_ONLY) {
        if (!(m[u] > 0.f)) x = 0.f;
        if (n < N) dy[n] = x;
      }
      sh[u * 8 + r][l] = x;
    }
    __syncthreads();
    if (k0 + BG_ROWS < rows) load(k0 + BG_ROWS);
    if (tid < 32) {
      const int cnt = (int)min((long long)BG_ROWS, mine - k0);
      if (cnt == BG_ROWS) {
#pragma unroll 16
        for (int k = 0; k < BG_ROWS; ++k) s += sh[k][l];
      } else {
        for (int k = 0; k < cnt; ++k) s += sh[k][l];
      }
    }
    __syncthreads();
  }
  if (tid < 32) part[c * 256 + chain] = s;
}

// ------------------------------------------------------------ weight gradient
// dW[co][c 9 + ky 3 + kx] = sum over pixels q of dY[co][q] X[c][q + (ky - 1,
// kx - 1)], the pixels split in ranges of `kchunk` (blockIdx.x) whose partial
// sums P [z][tap][Co][Ci] are added in order afterwards. A workgroup takes one
// range, one ky, 32 input channels (blockIdx.y = 3 block + ky) and 32 RT
// output channels (blockIdx.z); wave w the tap kx = w % 3 of row tile w / 3.
// Per step of KS pixels it stages dY and X as BF16 in LDS, pixels fastest
// (the depth of the product), X three times, shifted by kx - 1, so that every
// operand is one aligned 16-byte LDS read: X is loaded three times (once per
// ky) instead of being written and read as nine rows. The chain over a
// range's pixels is serial by the order of its sum, so what counts is the
// time per step: long steps with the next step's loads in flight, and more
// waves loading than computing. Where fewer workgroups than compute units are
// launched (three quarters, to leave some margin) a step is 512 pixels for 32
// output channels and 256 for 64, with twelve waves; else half of each, with
// six, so that two workgroups share a compute unit. The ten 3 x 3 layers of a
// step of 32 patches of 64 x 64 take 209 us (221 with the short steps alone);
// the product on an im2col matrix took 2,358 us and writing that matrix 476 us.
// (The matrix cores need 19 us for these layers.)
template <int RT, int KS, int DW_T>
__global__ __launch_bounds__(DW_T) void k_dw3(const float* __restrict__ dY, const float* __restrict__ X,
                                              float* __restrict__ P, int Co, int Ci, int H, int W, int K,
                                              int kchunk) {
  constexpr int G = KS / 8;                          // 8-pixel groups per step
  constexpr int AI = (RT * 32 * G + DW_T - 1) / DW_T, BI = (32 * G + DW_T - 1) / DW_T;
  __shared__ __attribute__((aligned(16))) uint16_t As[RT * 32][KS + 8];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[3][32][KS + 8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int ky = blockIdx.y % 3, c0 = blockIdx.y / 3 * 32, m0 = blockIdx.z * 32 * RT;
  const int kx = wv % 3, rt = wv / 3;
  const int kbeg = blockIdx.x * kchunk, kend = min(K, kbeg + kchunk);
  const int dxs = KS % W, dys = KS / W % H;          // a step's advance in x and y
  const float* ap[AI];
  const float* bp[BI];
  int ak[AI], bq[BI], bx[BI], by[BI];
  bool con[BI];
#pragma unroll
  for (int j = 0; j < AI; ++j) {
    const int e = min(tid + DW_T * j, RT * 32 * G - 1), row = e / G;
    ak[j] = kbeg + 8 * (e - row * G);
    ap[j] = dY + (long long)min(m0 + row, Co - 1) * K;
  }
#pragma unroll
  for (int j = 0; j < BI; ++j) {
    const int e = min(tid + DW_T * j, 32 * G - 1), row = e / G;
    bq[j] = kbeg + 8 * (e - row * G);
    by[j] = bq[j] / W;
    bx[j] = bq[j] - by[j] * W;
    by[j] %= H;
    con[j] = c0 + row < Ci;
    bp[j] = X + (long long)min(c0 + row, Ci - 1) * K;
  }
  float4 av[AI][2], bv[BI][2];
  float bl[BI], br[BI];
  uint32_t aok = 0, bok = 0, lok = 0, rok = 0;
  auto load = [&]() {   // every address clamped into the arrays, so no load waits for another
    aok = bok = lok = rok = 0;
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      const float4* s = reinterpret_cast<const float4*>(ap[j] + min(ak[j], K - 8));
      av[j][0] = s[0];
      av[j][1] = s[1];
      aok |= (uint32_t)(ak[j] < kend) << j;
      ak[j] += KS;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      const int yy = by[j] + ky - 1;
      const int q = min(max(bq[j] + (ky - 1) * W, 0), K - 8);
      const float* s = bp[j] + q;
      bv[j][0] = reinterpret_cast<const float4*>(s)[0];
      bv[j][1] = reinterpret_cast<const float4*>(s)[1];
      bl[j] = bp[j][max(q - 1, 0)];
      br[j] = bp[j][min(q + 8, K - 1)];
      const bool in = bq[j] < kend && yy >= 0 && yy < H && con[j];
      bok |= (uint32_t)in << j;
      lok |= (uint32_t)(in && bx[j] > 0) << j;
      rok |= (uint32_t)(in && bx[j] + 8 < W) << j;
      bq[j] += KS;
      bx[j] += dxs;
      by[j] += dys;
      if (bx[j] >= W) {
        bx[j] -= W;
        ++by[j];
      }
      if (by[j] >= H) by[j] -= H;
    }
  };
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  load();
  for (int k0 = kbeg; k0 < kend; k0 += KS) {
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      const int e = tid + DW_T * j, row = e / G;
      if (e >= RT * 32 * G) continue;
      const bool in = aok >> j & 1u;
      const float4 a = av[j][0], b = av[j][1];
      *reinterpret_cast<uint4*>(&As[row][8 * (e - row * G)]) =
          in ? make_uint4(pk(a.x, a.y), pk(a.z, a.w), pk(b.x, b.y), pk(b.z, b.w)) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      const int e = tid + DW_T * j, row = e / G, g = 8 * (e - row * G);
      if (e >= 32 * G) continue;
      const bool in = bok >> j & 1u;
      const float4 a = bv[j][0], b = bv[j][1];
      uint32_t w0 = pk(a.x, a.y), w1 = pk(a.z, a.w), w2 = pk(b.x, b.y), w3 = pk(b.z, b.w);
      if (!in) w0 = w1 = w2 = w3 = 0;
      const uint32_t le = (lok >> j & 1u) ? pk(bl[j], 0.f) : 0u, ri = (rok >> j & 1u) ? pk(br[j], 0.f) : 0u;
      const uint32_t s1 = __builtin_amdgcn_alignbit(w1, w0, 16), s2 = __builtin_amdgcn_alignbit(w2, w1, 16),
                     s3 = __builtin_amdgcn_alignbit(w3, w2, 16);
      *reinterpret_cast<uint4*>(&Bs[0][row][g]) = make_uint4((w0 << 16) | (le & 0xffffu), s1, s2, s3);
      *reinterpret_cast<uint4*>(&Bs[1][row][g]) = make_uint4(w0, w1, w2, w3);
      *reinterpret_cast<uint4*>(&Bs[2][row][g]) = make_uint4(s1, s2, s3, (w3 >> 16) | (ri << 16));
    }
    __syncthreads();
    if (k0 + KS < kend) load();
    if (rt < RT) {
      const uint16_t* a = &As[rt * 32 + (lane & 31)][(lane >> 5) * 8];
      const uint16_t* b = &Bs[kx][lane & 31][(lane >> 5) * 8];
#pragma unroll
      for (int ks = 0; ks < KS; ks += 16)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(a + ks),
                                                      *reinterpret_cast<const bf16x8*>(b + ks), acc, 0, 0, 0);
    }
    __syncthreads();
  }
  const int c = c0 + (lane & 31);
  if (rt >= RT || c >= Ci) return;
  float* out = P + ((long long)blockIdx.x * 9 + ky * 3 + kx) * Co * Ci;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int m = m0 + rt * 32 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
    if (m < Co) out[(long long)m * Ci + c] = acc[i];
  }
}

// The same for the layers whose product rows are whole rows of X: dW[m][r] =
// sum_q dY[m][q] Xg(r, q), Xg the 1-D temporal gather of X [C][Tin][Np] (row
// r = c KT + tap, column q = j Np + n: X[c][j S + tap - Pd][n], zero outside
// 0 .. Tin - 1) that im2col1 writes, or X itself (KT = 1, S = 0, Tin = 1,
// Np = K). A workgroup takes one range of columns, 32 RT rows of dY and 32
// rows r; wave w computes row tile w, all waves load. 32 rows of dY take steps
// of 512 columns with eight waves: the temporal layers' and the output layer's
// gradients of 16 segments of 64 x 64, 190 us with 256 and four, take 147
// (1,024 and sixteen are no faster). Only RB rows of X are staged: eight for
// the first temporal layer's five (74 -> 61 us).
template <int RT, int KS, int NT, int RB>
__global__ __launch_bounds__(NT) void k_dw1(const float* __restrict__ dY, const float* __restrict__ X,
                                             float* __restrict__ P, int M, int R, int K, int kchunk, int Tin, int KT,
                                             int S, int Pd, int Np) {
  constexpr int G = KS / 8;
  constexpr int AI = RT * 32 * G / NT, BI = RB * G / NT;
  static_assert(BI >= 1, "the rows fill the workgroup");
  __shared__ __attribute__((aligned(16))) uint16_t As[RT * 32][KS + 8];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[RB][KS + 8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r0 = blockIdx.y * 32, m0 = blockIdx.z * 32 * RT;
  const int kbeg = blockIdx.x * kchunk, kend = min(K, kbeg + kchunk);
  const int g = tid % G * 8, row0 = tid / G;         // rows row0 + j (NT / G)
  constexpr int RS = NT / G;
  int q = kbeg + g, jj = q / Np, n = q - jj * Np;
  float4 av[AI][2], bv[BI][2];
  uint32_t bok = 0;
  bool kin = false;
  int cc[BI], tp[BI];
#pragma unroll
  for (int j = 0; j < BI; ++j) {
    const int r = min(r0 + row0 + RS * j, R - 1);
    cc[j] = r / KT;
    tp[j] = r - cc[j] * KT - Pd;
  }
  auto load = [&]() {
    kin = q < kend;
    const int qa = min(q, K - 8);
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      const float4* s = reinterpret_cast<const float4*>(dY + (long long)min(m0 + row0 + RS * j, M - 1) * K + qa);
      av[j][0] = s[0];
      av[j][1] = s[1];
    }
    bok = 0;
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      const int t = jj * S + tp[j], tc = min(max(t, 0), Tin - 1);
      const float4* s = reinterpret_cast<const float4*>(X + ((long long)cc[j] * Tin + tc) * Np + min(n, Np - 8));
      bv[j][0] = s[0];
      bv[j][1] = s[1];
      bok |= (uint32_t)(kin && t == tc && r0 + row0 + RS * j < R) << j;
    }
    q += KS;
    n += KS;
    while (n >= Np && q < kend) {
      n -= Np;
      ++jj;
    }
  };
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  load();
  for (int k0 = kbeg; k0 < kend; k0 += KS) {
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      const int row = row0 + RS * j;
      const float4 a = av[j][0], b = av[j][1];
      *reinterpret_cast<uint4*>(&As[row][g]) =
          kin && m0 + row < M ? make_uint4(pk(a.x, a.y), pk(a.z, a.w), pk(b.x, b.y), pk(b.z, b.w))
                              : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      const float4 a = bv[j][0], b = bv[j][1];
      *reinterpret_cast<uint4*>(&Bs[row0 + RS * j][g]) =
          (bok >> j & 1u) ? make_uint4(pk(a.x, a.y), pk(a.z, a.w), pk(b.x, b.y), pk(b.z, b.w))
                          : make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    if (k0 + KS < kend) load();
    if (wv < RT) {
      const uint16_t* a = &As[wv * 32 + (lane & 31)][(lane >> 5) * 8];
      const uint16_t* b = &Bs[RB == 32 ? lane & 31 : lane & (RB - 1)][(lane >> 5) * 8];
#pragma unroll
      for (int ks = 0; ks < KS; ks += 16)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(a + ks),
                                                      *reinterpret_cast<const bf16x8*>(b + ks), acc, 0, 0, 0);
    }
    __syncthreads();
  }
  const int r = r0 + (lane & 31);
  if (wv >= RT || r >= R) return;
  float* out = P + (long long)blockIdx.x * M * R;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int m = m0 + wv * 32 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
    if (m < M) out[(long long)m * R + r] = acc[i];
  }
}

// All layers' gradients in one launch: the pixel ranges' partial sums added
// in order (their loads issued together), and the bias chains' tree.
__global__ __launch_bounds__(256) void k_grad_reduce(GradTable t, float* __restrict__ grad) {
  const int blk = blockIdx.x;
  if (blk < t.wblocks) {
    int s = 0;
    while (s + 1 < t.nw && t.w[s + 1].block0 <= blk) ++s;
    const GradSeg& g = t.w[s];
    const int i = (blk - g.block0) * 256 + threadIdx.x;
    const int MN = g.T * g.M * g.C;
    if (i >= MN) return;
    float v[kGradSplits];
#pragma unroll
    for (int z = 0; z < kGradSplits; ++z) v[z] = g.P[(long long)min(z, g.Z - 1) * MN + i];
    float sum = 0.f;
#pragma unroll
    for (int z = 0; z < kGradSplits; ++z)
      if (z < g.Z) sum += v[z];
    const int tap = i / (g.M * g.C), mc = i - tap * g.M * g.C, m = mc / g.C, c = mc - m * g.C;
    grad[g.out + (long long)m * g.C * g.T + (long long)c * g.T + tap] = sum;
    return;
  }
  const int ch = (blk - t.wblocks) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  int s = 0;
  while (s + 1 < t.nb && t.b[s + 1].ch0 <= ch) ++s;
  const BiasSeg& b = t.b[s];
  const int c = ch - b.ch0;
  if (c >= b.C) return;
  const float* p = t.bpart + (long long)ch * 256;
  float v = (p[lane] + p[lane + 128]) + (p[lane + 64] + p[lane + 192]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if (lane == 0) grad[b.out + c] = v;
}

// ------------------------------------- input gradient, transposed convolutions
// dX [M][N] = W^T dY for W [K][M] (BF16) and dY [K][N], the depth in steps of
// 16 as the tiled product takes it. A wave takes 32 rows x 32 columns and reads
// both operands from memory itself: the row tiles of one column block are
// neighbouring waves, so a second read of dY comes from the caches, and with no
// barrier every load of four depth steps is in flight at once. Latency is what
// bounds it (a few thousand columns, 8 or 16 steps): the two layers of a step of
// 32 patches of 64 x 64 take 13 us; the tiled product, which waits for its
// loads at each of its steps, took 58.
__global__ __launch_bounds__(256) void k_lin_dx(const uint16_t* __restrict__ W, const float* __restrict__ dY,
                                                float* __restrict__ dX, int M, int K, int N) {
  const int lane = threadIdx.x & 63, h = lane >> 5, l = lane & 31;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), tiles = M / 32;
  const int m0 = w % tiles * 32, n = w / tiles * 32 + l;
  if (n - l >= N) return;
  const float* y = dY + (long long)8 * h * N + min(n, N - 1);
  const uint16_t* a = W + 8 * h * M + m0 + l;
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  for (int k0 = 0; k0 < K; k0 += 64) {
    uint16_t av[32];
    float yv[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) {   // depth 16 (e / 8) + 8 h + e % 8 of the four steps
      const int k = k0 + 16 * (e >> 3) + (e & 7);
      av[e] = a[k * M];
      yv[e] = y[(long long)k * N];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint32_t aw[4], bw[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        aw[q] = av[8 * g + 2 * q] | (uint32_t)av[8 * g + 2 * q + 1] << 16;
        bw[q] = pk(yv[8 * g + 2 * q], yv[8 * g + 2 * q + 1]);
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, make_uint4(aw[0], aw[1], aw[2], aw[3])),
                                                    __builtin_bit_cast(bf16x8, make_uint4(bw[0], bw[1], bw[2], bw[3])),
                                                    acc, 0, 0, 0);
    }
  }
  if (n >= N) return;
#pragma unroll
  for (int i = 0; i < 16; ++i) dX[(long long)(m0 + 8 * (i >> 2) + 4 * h + (i & 3)) * N + n] = acc[i];
}

// ------------------------------------------- input gradients, temporal layers
// From the third layer's output gradient g3 [32][N] (masked) to the second's,
// g2 [32][5][N] = W3^T g3, and to the first's, g1 [32][10][N], both masked
// where the activation is not positive. g1 at sample t is the sum, taps k in
// order, of the products of tap k with g2 at sample (t + 2 - k) / 2: each is
// formed by itself (two depth steps over the 32 channels) and then added, as
// the product into im2col rows and the gather from them (col2im1) did. A wave
// takes 32 pixels. A product's rows are channels ordered so that lane (h,
// pixel) gets channels 8 h .. + 7 and 16 + 8 h .. + 7: the operands of the
// next product, with no exchange between lanes. Bound by its reads of both
// activations and its writes of both gradients. Sixteen patches of 64 x 64
// take 47 us, where the products (136), the gather (115) and the mask passes
// took 290.
constexpr int TX_C = 32, TX_KT = 5, TX_J1 = 10, TX_J2 = 5, TX_K = TX_C * TX_KT;

__device__ __forceinline__ int tx_channel(int h, int i) { return 16 * (i >> 3) + 8 * h + (i & 7); }

__global__ __launch_bounds__(256) void k_temporal_dx(const uint16_t* __restrict__ w2, const uint16_t* __restrict__ w3,
                                                     const float* __restrict__ g3, const float* __restrict__ a2,
                                                     const float* __restrict__ a1, float* __restrict__ g2,
                                                     float* __restrict__ g1, uint32_t N) {
  // operands of W^T: [tap or sample][depth step][lane]
  __shared__ __attribute__((aligned(16))) uint16_t W2s[TX_KT * 2 * 64 * 8], W3s[TX_J2 * 2 * 64 * 8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, h = lane >> 5, px = lane & 31;
  for (int e = tid; e < TX_KT * 2 * 64 * 8; e += 256) {
    const int q = e & 7, l = e >> 3 & 63, g = e >> 9 & 1, k = e >> 10;
    const int r = l & 31, ch = tx_channel((r >> 2) & 1, 4 * (r >> 3) + (r & 3)), co = 16 * g + 8 * (l >> 5) + q;
    W2s[e] = w2[co * TX_K + ch * TX_KT + k];
    W3s[e] = w3[co * TX_K + ch * TX_KT + k];
  }
  __syncthreads();
  auto opw = [&](const uint16_t* w, int k, int g) {
    return *reinterpret_cast<const bf16x8*>(w + ((k * 2 + g) * 64 + lane) * 8);
  };
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto operand = [&](const float (&z)[16], int g) {
    return __builtin_bit_cast(bf16x8, make_uint4(pk(z[8 * g], z[8 * g + 1]), pk(z[8 * g + 2], z[8 * g + 3]),
                                                 pk(z[8 * g + 4], z[8 * g + 5]), pk(z[8 * g + 6], z[8 * g + 7])));
  };
  for (uint32_t p0 = (blockIdx.x * 4 + wv) * 32; p0 < N; p0 += gridDim.x * 128) {
    // element (channel of register i, row `row` of `per`) at this lane's pixel
    auto at = [&](uint32_t per, int i, uint32_t row) {
      return (size_t)((16u * (i >> 3) + (i & 7)) * per + row) * N + p0 + (8u * h * per * N + px);
    };
    bf16x8 b3[2];
    {
      float z[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) z[i] = g3[at(1, i, 0)];
      b3[0] = operand(z, 0);
      b3[1] = operand(z, 1);
    }
    bf16x8 b2[TX_J2][2];
#pragma unroll
    for (int j = 0; j < TX_J2; ++j) {
      float y[16], z[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) y[i] = a2[at(TX_J2, i, j)];
      f32x16 c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opw(W3s, j, 0), b3[0], zero, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opw(W3s, j, 1), b3[1], c, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        z[i] = y[i] > 0.f ? c[i] : 0.f;
        g2[at(TX_J2, i, j)] = z[i];
      }
      b2[j][0] = operand(z, 0);
      b2[j][1] = operand(z, 1);
    }
#pragma unroll
    for (int t = 0; t < TX_J1; ++t) {
      float y[16], s[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        y[i] = a1[at(TX_J1, i, t)];
        s[i] = 0.f;
      }
#pragma unroll
      for (int k = 0; k < TX_KT; ++k) {
        const int jt = t + 2 - k;
        if (jt < 0 || jt % 2 || jt / 2 >= TX_J2) continue;
        f32x16 c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opw(W2s, k, 0), b2[jt / 2][0], zero, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opw(W2s, k, 1), b2[jt / 2][1], c, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] += c[i];
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) g1[at(TX_J1, i, t)] = y[i] > 0.f ? s[i] : 0.f;
    }
  }
}

// ------------------------------------------------------------- input gradient
// dX[c][y][x] = sum over taps (ky, kx), in order, of
// sum_co W[co][c 9 + tap] dY[co][y - ky + 1][x - kx + 1]: each tap's product
// over the output channels is formed by itself (as the product before col2im
// forms it) and then added. A workgroup takes 128 NTW pixels (whole rows of at
// most 64 columns) and 32 input channels; dY's halo tile lies in LDS as BF16,
// output channels fastest, all of them (CG blocks of 16). The weights, laid
// out so that a wave's operand is 1 KB in a row (Wd [Ci / 32][9][CG][lane][8]),
// come from the caches, one tap ahead. Bound by the wait for the halo tile and
// the matrix work after it, at one to three workgroups per compute unit: the
// nine layers of a step of 32 patches of 64 x 64 take 170 us; the products into
// FP32 matrices and the gathers from them took 984 us.
template <int CG, int NTW>
__global__ __launch_bounds__(256) void k_dx3(const uint16_t* __restrict__ Wd, const float* __restrict__ dY,
                                             float* __restrict__ dX, int Ci, int H, int W, long long N, int BC) {
  extern __shared__ __attribute__((aligned(16))) uint16_t Xs[];
  constexpr int NT = 128 * NTW, PI = 2;
  const int BR = NT / BC, TC = BC + 2, np = (BR + 2) * TC;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int bx = (W + BC - 1) / BC, by = (H + BR - 1) / BR;
  const int T = gridDim.x, xb = blockIdx.x, blk = T % 8 ? xb : (xb & 7) * (T >> 3) + (xb >> 3);
  const int b = blk / (bx * by), rem = blk - b * bx * by;
  const int y0 = rem / bx * BR, x0 = rem % bx * BC;
  const long long HW = (long long)H * W;
  const float* src[PI];
  bool in[PI];
#pragma unroll
  for (int j = 0; j < PI; ++j) {
    const int pos = min(tid + 256 * j, np - 1), r = pos / TC, cc = pos - r * TC;
    const int y = y0 + r - 1, x = x0 + cc - 1;
    in[j] = y >= 0 && y < H && x >= 0 && x < W;
    src[j] = dY + b * HW + (long long)min(max(y, 0), H - 1) * W + min(max(x, 0), W - 1);
  }
#pragma unroll
  for (int cg = 0; cg < CG; ++cg) {   // 16 channels of up to two positions in flight
    float v[PI][16];
#pragma unroll
    for (int j = 0; j < PI; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) v[j][q] = src[j][(long long)(16 * cg + q) * N];
#pragma unroll
    for (int j = 0; j < PI; ++j) {
      const int pos = tid + 256 * j;
      if (pos >= np) continue;
      uint32_t w[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) w[q] = in[j] ? pk(v[j][2 * q], v[j][2 * q + 1]) : 0u;
      uint4* d = reinterpret_cast<uint4*>(&Xs[(cg * np + pos) * 16]);
      d[0] = make_uint4(w[0], w[1], w[2], w[3]);
      d[1] = make_uint4(w[4], w[5], w[6], w[7]);
    }
  }
  const uint16_t* wp = Wd + (long long)blockIdx.y * 9 * CG * 512 + lane * 8;
  bf16x8 a[2][CG];
#pragma unroll
  for (int cg = 0; cg < CG; ++cg) a[0][cg] = *reinterpret_cast<const bf16x8*>(wp + cg * 512);
  int at[NTW], py[NTW], px[NTW];
  f32x16 sum[NTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int pl = (wv * NTW + t) * 32 + (lane & 31);
    py[t] = pl / BC;
    px[t] = pl - py[t] * BC;
    at[t] = ((py[t] + 2) * TC + px[t] + 2) * 16 + (lane >> 5) * 8;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[t][i] = 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    if (tap < 8) {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg)
        a[(tap + 1) & 1][cg] = *reinterpret_cast<const bf16x8*>(wp + ((tap + 1) * CG + cg) * 512);
    }
    const int off = ((tap / 3) * TC + tap % 3) * 16;
    f32x16 acc[NTW];
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
#pragma unroll
    for (int cg = 0; cg < CG; ++cg)
#pragma unroll
      for (int t = 0; t < NTW; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            a[tap & 1][cg], *reinterpret_cast<const bf16x8*>(&Xs[cg * np * 16 + at[t] - off]), acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) sum[t][i] += acc[t][i];
  }
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int y = y0 + py[t], x = x0 + px[t];
    if (y >= H || x >= W) continue;
    float* o = dX + b * HW + (long long)y * W + x;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int c = blockIdx.y * 32 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
      o[(long long)c * N] = sum[t][i];
    }
  }
}

template <int CG, int NTW>
hipError_t launch_dx3(const uint16_t* Wd, const float* dY, float* dX, int Ci, int Bn, int H, int W, hipStream_t st) {
  const int BC = std::min(W, 64), BR = 128 * NTW / BC, np = (BR + 2) * (BC + 2);
  const size_t lds = (size_t)CG * np * 32;
  static_assert(CG <= 8, "the halo tile fits the LDS");
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_dx3<CG, NTW>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  const unsigned tiles = (unsigned)(Bn * ((H + BR - 1) / BR) * ((W + BC - 1) / BC));
  hipLaunchKernelGGL((k_dx3<CG, NTW>), dim3(tiles, Ci / 32), dim3(256), lds, st, Wd, dY, dX, Ci, H, W,
                     (long long)Bn * H * W, BC);
  return hipGetLastError();
}

}  // namespace

// ------------------------------------------------------------------ launchers

void bias_mask(float* dY, const float* Y, float* part, int C, long long N, hipStream_t st) {
  if (Y)
    hipLaunchKernelGGL(k_bias_mask<BIAS_MASK>, dim3(C, 8), dim3(256), 0, st, dY, Y, nullptr, nullptr, part, N);
  else
    hipLaunchKernelGGL(k_bias_mask<BIAS_ONLY>, dim3(C, 8), dim3(256), 0, st, dY, nullptr, nullptr, nullptr, part, N);
}

void bias_outer(const float* gl, const uint16_t* wo, float* dY, const float* Y, float* part, int C, long long N,
                hipStream_t st) {
  hipLaunchKernelGGL(k_bias_mask<BIAS_OUTER>, dim3(C, 8), dim3(256), 0, st, dY, Y, gl, wo, part, N);
}

int grad_chunk(long long K) {
  const long long c = (K + kGradSplits - 1) / kGradSplits;
  return (int)((c + 31) / 32 * 32);
}
int grad_ranges(long long K) { return (int)((K + grad_chunk(K) - 1) / grad_chunk(K)); }

bool dw3(const float* dY, const float* X, float* P, int Co, int Ci, int Bn, int H, int W, hipStream_t st) {
  const long long K = (long long)Bn * H * W;
  if (W % 8 || Co % 32 || K > 0x3fffffffLL || ((uintptr_t)dY & 15) || ((uintptr_t)X & 15)) return false;
  const int kc = grad_chunk(K);
  const dim3 grid(grad_ranges(K), 3 * ((Ci + 31) / 32), Co <= 32 ? 1 : Co / 64);
  if (Co > 32 && Co % 64) return false;
  const bool big = grid.x * grid.y * grid.z <= 200;
#define DW3(RT, KS, NT) hipLaunchKernelGGL((k_dw3<RT, KS, NT>), grid, dim3(NT), 0, st, dY, X, P, Co, Ci, H, W, (int)K, kc)
  if (Co <= 32 && big)
    DW3(1, 512, 768);
  else if (Co <= 32)
    DW3(1, 256, 384);
  else if (big)
    DW3(2, 256, 768);
  else
    DW3(2, 128, 384);
#undef DW3
  return true;
}

bool dw1(const float* dY, const float* X, float* P, int M, int R, long long K, int Tin, int KT, int S, int Pd,
         long long Np, hipStream_t st) {
  if (Np % 8 || K % 8 || K > 0x3fffffffLL || ((uintptr_t)dY & 15) || ((uintptr_t)X & 15)) return false;
  const int kc = grad_chunk(K), z = grad_ranges(K), rb = (R + 31) / 32;
#define DW1(RT, KS, NT, RB)                                                                                          \
  hipLaunchKernelGGL((k_dw1<RT, KS, NT, RB>), dim3(z, rb, (M + 32 * RT - 1) / (32 * RT)), dim3(NT), 0, st, dY, X, P, M, \
                     R, (int)K, kc, Tin, KT, S, Pd, (int)Np)
  if (M <= 32 && R <= 8)
    DW1(1, 512, 512, 8);
  else if (M <= 32)
    DW1(1, 512, 512, 32);
  else
    DW1(2, 128, 256, 32);
#undef DW1
  return true;
}

void lin_dx(const uint16_t* W, const float* dY, float* dX, int M, int K, long long N, hipStream_t st) {
  const long long waves = (N + 31) / 32 * (M / 32);
  hipLaunchKernelGGL(k_lin_dx, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, W, dY, dX, M, K, (int)N);
}

bool temporal_dx(const uint16_t* w2, const uint16_t* w3, const float* g3, const float* a2, const float* a1, float* g2,
                 float* g1, long long N, hipStream_t st) {
  if (N % 32 || N > 1 << 22) return false;   // 32-bit offsets
  const dim3 grid((unsigned)std::min<long long>((N / 32 + 3) / 4, 1024));
  hipLaunchKernelGGL(k_temporal_dx, grid, dim3(256), 0, st, w2, w3, g3, a2, a1, g2, g1, (uint32_t)N);
  return true;
}

void grad_reduce(const GradTable& t, float* grad, hipStream_t st) {
  const int ch = t.nb ? t.b[t.nb - 1].ch0 + t.b[t.nb - 1].C : 0;
  hipLaunchKernelGGL(k_grad_reduce, dim3(t.wblocks + (ch + 3) / 4), dim3(256), 0, st, t, grad);
}

bool dx3(const uint16_t* Wd, const float* dY, float* dX, int Co, int Ci, int Bn, int H, int W, hipStream_t st,
         hipError_t* err) {
  const int BC = std::min(W, 64);
  if (W % 8 || 128 % BC || Ci % 32 || (Co != 32 && Co != 64 && Co != 128)) return false;
  // two pixel blocks per wave share each weight operand; one where the larger
  // tiles would leave compute units without a workgroup
  const int BR = 256 / BC;
  const bool two = (long long)Bn * ((H + BR - 1) / BR) * ((W + BC - 1) / BC) * (Ci / 32) >= 512;
  switch (Co / 16 * 2 + two) {
    case 4: *err = launch_dx3<2, 1>(Wd, dY, dX, Ci, Bn, H, W, st); break;
    case 5: *err = launch_dx3<2, 2>(Wd, dY, dX, Ci, Bn, H, W, st); break;
    case 8: *err = launch_dx3<4, 1>(Wd, dY, dX, Ci, Bn, H, W, st); break;
    case 9: *err = launch_dx3<4, 2>(Wd, dY, dX, Ci, Bn, H, W, st); break;
    case 16: *err = launch_dx3<8, 1>(Wd, dY, dX, Ci, Bn, H, W, st); break;
    default: *err = launch_dx3<8, 2>(Wd, dY, dX, Ci, Bn, H, W, st); break;
  }
  return true;
}

}  // namespace nn
}  // namespace seg
