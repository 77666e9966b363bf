// Streaming segment-summary kernel: one pass over the uint16 video computes,
// per 50-frame segment and pixel,
//   S_i  temporal mean (Eq. 1),
//   T_i  max minus median over time of the Gaussian-smoothed video (Eq. 2),
//   D_i  mean of max(0, median - smoothed value) (noise-scale term),
//   U_i, P_i  sums of reference-subtracted values and of their products with
//        the right, lower, lower-right and lower-left neighbours (pooled
//        co-moments of the correlation image).
//
// Work decomposition: one workgroup of 256 threads per (64 x 16 pixel tile,
// segment). Per frame the tile plus a 12-pixel halo (88 x 40) is staged in
// LDS as d = V - R, where R is a per-pixel integer reference (the median of
// the segment's first three frames). Subtracting R leaves T, D and the
// centred co-moments unchanged but keeps the smoothed values small, so the
// per-pixel window can be held in FP32 without losing the precision the
// event threshold needs.
//
// The separable smoothing is a banded product, 16 outputs from 40 inputs, and
// runs on INT8 MFMA in fixed point: d (scaled by a power of two) is two signed
// bytes and a weight (times 2^30) four, so the vertical pass is eight byte
// products, exact in INT32; its result, rounded to 20 fraction bits, is four
// bytes, and the horizontal pass takes the thirteen byte products of 2^-27
// and more of the largest. One FP64 sum per value restores it, exact but for
// that rounding, and rounds it to FP32. The error of T and D is no larger than
// that of FP64 sums with an FP32 intermediate (measured against FP64 over
// pushes, whole recordings and served mixes: 2.6e-8 to 3.9e-8, with FP64 sums
// 2.6e-8 to 4.1e-8). A frame whose values do not fit the scale (|d| above
// 2,000 divided by the power of two, which leaves four times the range of the
// first three frames where that fits) takes the general path from its chunk
// of ten frames on: FP64 sums over 25 taps in both passes.
//
// What bounds it: vector instructions of the two waves that a SIMD holds (the
// FP32 window, 200 values of a thread, allows no third), then the chain from
// staging through both passes where a launch has one workgroup per compute
// unit. Hence 16-bit arithmetic while staging, byte planes laid out as the
// matrix operands read them, and one barrier per frame with the three steps
// of three frames between two. Measured, from FP64 sums and two barriers per
// frame (which also read a width that is no multiple of four pixel by pixel):
// 64 x 64 x 50 99 -> 80 us, 450 x 138 x 500 561 -> 168 us, four recordings of
// 500 frames in one launch (128 x 128 to 512 x 512) 1,520 -> 1,000 us.
// With two barriers and single buffers the same products took 92, 205 and
// 1,620 us. Frames that all take the general path: 256 x 256 x 1,600 604 ->
// 680 us with values over the whole 16-bit range, 626 us with one bright frame
// per segment in every tile.
//
// Every thread owns 4 adjacent pixels of one tile row and keeps their 50
// smoothed values in VGPRs (40) and a per-thread LDS slot (the chunk being
// filled); after the segment a compare-exchange network gives the median, the
// maximum and the 25 smallest values.
#include "seg_kernels.h"
#include "selnet_gen.h"

namespace seg {
namespace {

constexpr int L = kSegLen;
constexpr int RAD = kMaxRadius;
constexpr int NTAP = 2 * RAD + 1;
constexpr int TW = 64, TH = 16;
constexpr int DW = TW + 2 * RAD;     // 88 staged columns
constexpr int DH = TH + 2 * RAD;     // 40 staged rows
constexpr int NT = 256;
constexpr int NPX = 4;               // pixels per thread
constexpr int CH = 10;               // frames per unrolled chunk
constexpr int NCH = L / CH;          // 5 chunks per segment
static_assert(L % CH == 0, "chunking");

struct KParams {
  const uint16_t* src0;
  const uint16_t* src1;
  long long n0;
  int H, W;
  int seg0, nseg;
  float *T, *S, *D, *U, *P;
  long long plane;
  double w[NTAP];
};

struct BatchSlot {
  KParams p;
  int ntile;   // tiles per segment
  int item0;   // first work item of this slot
};

struct BatchTable {
  int nslots;
  int total;   // work items over all slots
  int pad[2];
  BatchSlot slot[kMaxBatch];
};

__device__ __forceinline__ int reflect(int j, int n) {
  const int m = 2 * n;
  j %= m;
  if (j < 0) j += m;
  return j >= n ? m - 1 - j : j;
}

// LDS-only workgroup barrier: waits for this wave's LDS traffic, not for its
// outstanding global loads, so the next frame's prefetch stays in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Vertical pass for one (column, 8-row) task: U rows 8h..8h+7 of column c,
// streaming the 32 staged rows once.
constexpr int VROWS = 8;
constexpr int NVT8 = DW * (TH / VROWS);   // 176 tasks, one round
static_assert(NVT8 <= NT, "one vertical round");

__device__ __forceinline__ void vtask8(int q, const float* __restrict__ Dl,
                                       float* __restrict__ Ul, const KParams& p) {
  const int c = q % DW;
  const int h = q / DW;
  const float* col = Dl + h * VROWS * DW + c;
  double acc[VROWS];
#pragma unroll
  for (int o = 0; o < VROWS; ++o) acc[o] = 0.0;
#pragma unroll
  for (int j = 0; j < NTAP + VROWS - 1; ++j) {
    const double x = (double)col[j * DW];
#pragma unroll
    for (int o = 0; o < VROWS; ++o)
      if (j - o >= 0 && j - o < NTAP) acc[o] = fma(p.w[j - o], x, acc[o]);
  }
  float* out = Ul + h * VROWS * DW + c;
#pragma unroll
  for (int o = 0; o < VROWS; ++o) out[o * DW] = (float)acc[o];
}

typedef int i4 __attribute__((ext_vector_type(4)));
typedef short s2 __attribute__((ext_vector_type(2)));
typedef unsigned short u2 __attribute__((ext_vector_type(2)));
typedef uint32_t px4 __attribute__((ext_vector_type(2), aligned(2)));   // four pixels at any pixel's address
typedef const __attribute__((address_space(1))) uint16_t* gpixels;
typedef const __attribute__((address_space(1))) char* gbytes;

// Staging: thread cq 10 + rq takes the 4 x 4 pixels of rows 4 rq .. and
// columns 4 cq .. of the staged region, so that the bytes of four rows of a
// column are one LDS word. Four neighbouring columns, folded at the frame's
// border in whatever way, lie in four contiguous source columns; one 8-byte
// load and a byte permutation fetch them.
constexpr int QR = DH / 4, QC = DW / 4;   // 10 x 22 items
static_assert(QR * QC <= NT, "one item per thread");
constexpr int NB = 6;                     // blocks of 16 staged columns (the last one half used)
constexpr int NV = 7;                     // blocks of 16 columns of the intermediate that are read
constexpr int PR = TH + 4;                // staged rows 12 .. 31 ..
constexpr int PS = TW / 2 + 4;            // .. and columns 8 .. 79 as 16-bit pairs: words per row
constexpr int kFrac = 20;                 // fraction bits of the intermediate
constexpr int kRange = 2000;              // |d| 2^e at most: 2000 * 2^20 and its byte carries are below 2^31

struct Smem {
  // Operands lie as the lanes of a wave read them, 16 bytes each in a row:
  // [block][16 rows][column] low and high bytes of d 2^e, and [block][row] the
  // bytes of 16 columns of the intermediate, lowest byte first. Even and odd
  // frames have their own.
  union {
    uint32_t b[2][2][NB * 3 * 16 * 4];
    float d[DH * DW];          // general path: d
  } in;
  union {
    uint32_t b[2][4][NV * 16 * 4];
    float u[TH * DW];          // general path: the intermediate
  } mid;
  uint32_t d16[2][PR * PS];
  uint32_t r16[TH * TW / 2];   // R of the tile's own pixels
  float4 Wl[CH * NT];
  int bad[NCH];                // a frame staged in this chunk does not fit the scale
  int cut;                     // a difference may not have fit 16 bits
  int top[4];
};
static_assert(sizeof(Smem) <= 80 * 1024, "two workgroups per compute unit");

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}

// 16 output values from 40 inputs along the depth of a 16 x 16 x 64 product:
// lane l holds, for output l % 16, the four bytes (lowest first) of the
// weights of inputs 16 (l / 16) .. + 15: w[input - output] 2^30.
__device__ __forceinline__ void band(const double* __restrict__ w, int lane, i4 (&wb)[4]) {
  const int m = lane & 15, k0 = 16 * (lane >> 4);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int tap = k0 + 4 * j + u - m;
      const double x = tap >= 0 && tap < NTAP ? w[min(max(tap, 0), NTAP - 1)] : 0.0;
      // signed bytes: a byte above 127 is taken off and carried to the next
      q[u] = ((uint32_t)(int)__builtin_rint(x * 1073741824.0) + 0x00808080u) ^ 0x00808080u;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t sel = 0x0c0c0000u | (uint32_t)(4 + b) << 8 | (uint32_t)b;   // byte b of both, zeros above
      wb[b][j] = (int)perm(perm(q[3], q[2], sel), perm(q[1], q[0], sel), 0x05040100u);
    }
  }
}

// One (segment sl, tile) work item of one recording. RARE tells the compiler
// how seldom the general path is (never, or one in twenty), and so whose values
// it keeps in registers: the batch kernel, short of them for its loop over
// items, takes 1,000 us with the first and 1,080 with the second at the mix
// above; the other kernel 166 and 168 us at 450 x 138 x 500, but 787 and 680 us
// where every frame takes the general path.
template <bool RARE>
__device__ __forceinline__ void block_body(const KParams& p, int sl, int tile, Smem& sm) {
  float4* Wl = sm.Wl;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = p.W, H = p.H;
  const int tiles_x = (W + TW - 1) / TW;
  const int ty0 = (tile / tiles_x) * TH;
  const int tx0 = (tile % tiles_x) * TW;
  const long long M = (long long)H * W;

  // Frames as global memory: pointers that come from the slot table would be
  // read with generic loads, which an LDS barrier waits for.
  const long long fbase = (long long)sl * L;
  const uint16_t *src0 = p.src0, *src1 = p.src1;
  const long long n0 = p.n0;
  auto frame = [&](int t) -> gpixels {
    const long long f = fbase + t;
    return (gpixels)(f < n0 ? src0 + f * M : src1 + (f - n0) * M);
  };

  // ---- staging geometry
  const bool loads = tid < QR * QC;
  const int cq = loads ? tid / QR : 0, rq = loads ? tid - cq * QR : 0;
  unsigned off[4];         // byte offset of the first of the four source columns, per row
  uint32_t sel01, sel23;   // bytes of columns 0, 1 and 2, 3 among the eight loaded
  {
    int c[4], lo = W;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      c[i] = reflect(tx0 - RAD + 4 * cq + i, W);
      lo = min(lo, c[i]);
    }
    lo = max(min(lo, W - 4), 0);
    auto bytes = [&](int i) { return (uint32_t)(2 * (c[i] - lo)) * 0x0101u + 0x0100u; };
    sel01 = bytes(0) | bytes(1) << 16;
    sel23 = bytes(2) | bytes(3) << 16;
#pragma unroll
    for (int k = 0; k < 4; ++k) off[k] = 2u * (unsigned)(reflect(ty0 - RAD + 4 * rq + k, H) * W + lo);
  }
  // four rows of four pixels, as loaded
  auto load = [&](gpixels fr, uint2 (&v)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const px4 w = *(const __attribute__((address_space(1))) px4*)((gbytes)fr + off[k]);
      v[k] = make_uint2(w.x, w.y);
    }
  };
  // frames narrower than four columns have the (up to three) pixels of the
  // row one by one, and take the general path
  auto load_any = [&](gpixels fr, uint2 (&v)[4]) {
    if (W >= 4) {
      load(fr, v);
      return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      gpixels r = (gpixels)((gbytes)fr + off[k]);
      const uint32_t a = r[0], b = r[min(1, W - 1)], c = r[min(2, W - 1)];
      v[k] = make_uint2(a | b << 16, c);
    }
  };
  auto pair = [&](uint2 v, uint32_t sel) { return perm(v.y, v.x, sel); };
  const bool centre = loads && rq >= RAD / 4 && rq < (RAD + PR) / 4 && cq >= 2 && cq < 2 + PS / 2;

  // ---- per-pixel reference: median of the segment's first three frames, and
  // the scale from the largest |V - R| among them
  uint32_t R[4][2];
  int e;          // d is scaled by 2^e
  bool general;   // the FP64 path
  {
    uint2 f0[4], f1[4], f2[4];
    load_any(frame(0), f0);
    load_any(frame(1), f1);
    load_any(frame(2), f2);
    u2 top = {0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t s = h ? sel23 : sel01;
        const u2 a = __builtin_bit_cast(u2, pair(f0[k], s)), b = __builtin_bit_cast(u2, pair(f1[k], s)),
                 c = __builtin_bit_cast(u2, pair(f2[k], s));
        const u2 lo = __builtin_elementwise_min(a, b), hi = __builtin_elementwise_max(a, b);
        const u2 r = __builtin_elementwise_max(lo, __builtin_elementwise_min(hi, c));
        // the largest and the smallest of the three, against the median
        const u2 mx = __builtin_elementwise_max(hi, c), mn = __builtin_elementwise_min(lo, c);
        top = __builtin_elementwise_max(top, __builtin_elementwise_max((u2)(mx - r), (u2)(r - mn)));
        R[k][h] = __builtin_bit_cast(uint32_t, r);
      }
    if (loads && rq >= RAD / 4 && rq < (RAD + TH) / 4 && cq >= RAD / 4 && cq < (RAD + TW) / 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<uint2*>(&sm.r16[(4 * rq + k - RAD) * (TW / 2) + 2 * cq - RAD / 2]) = make_uint2(R[k][0], R[k][1]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      R[k][0] ^= 0x80008000u;   // as the signed subtraction below wants it
      R[k][1] ^= 0x80008000u;
    }
    int t = max((int)top.x, (int)top.y);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t = max(t, __shfl_xor(t, o, 64));
    if (lane == 0) sm.top[wv] = t;
    if (tid < NCH) sm.bad[tid] = 0;
    if (tid == 0) sm.cut = 0;
    __syncthreads();
    t = max(max(max(sm.top[0], sm.top[1]), max(sm.top[2], sm.top[3])), 1);
    general = W < 4 || __builtin_amdgcn_readfirstlane(t) > kRange;
    e = 0;
    while (e < 7 && 4 * t << (e + 1) <= kRange) ++e;
    e = __builtin_amdgcn_readfirstlane(e);
  }
  const short lim = (short)(kRange >> e);

  // ---- thread-owned pixels: tile row hy, columns hx0 .. hx0+3 (the layout of
  // the horizontal product's result)
  const int hy = lane & 15, q = lane >> 4;
  const int hx0 = 16 * wv + 4 * q;

  i4 wb[4];
  band(p.w, lane, wb);

  // 40 of the 50 window values live in VGPRs (chunks 0..3); the chunk being
  // filled lives in a per-thread LDS slot, so the frame loop needs no
  // compile-time frame index. The chunk loop is unrolled, so a completed
  // chunk c moves once into its own registers win[c].
  float win[NCH - 1][CH][NPX];
  // Co-moment sums: whole numbers, exact in FP32.
  float Uacc[NPX], Pacc[5][NPX];

  // (a) stage d = V - R of the tile and its halo from the prefetched frame
  uint2 pf[4];
  const int to = (((cq >> 2) * 3 + (rq >> 2)) * 16) * 4 + (rq & 3);
  const int tc = 4 * (cq & 3) + (rq >> 2);   // columns turned by the row block: fewer lanes on one bank
  auto stage = [&](int buf, int c) {
    if (!loads) return;
    s2 d[4][2];
    u2 over = {0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const s2 v = __builtin_bit_cast(s2, pair(pf[k], h ? sel23 : sel01) ^ 0x80008000u);
        d[k][h] = __builtin_elementwise_sub_sat(v, __builtin_bit_cast(s2, R[k][h]));
        over = __builtin_elementwise_max(over, __builtin_bit_cast(u2, (s2)(d[k][h] + lim)));   // 0 .. 2 lim in range
      }
    const int far = max((int)over.x, (int)over.y);
    if (far > 2 * lim) {
      sm.bad[c] = 1;
      if (far >= 32767 + lim) sm.cut = 1;   // (or below the range by any amount)
    }
    if (centre) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<uint2*>(&sm.d16[buf][(4 * rq + k - RAD) * PS + 2 * cq - 4]) =
            make_uint2(__builtin_bit_cast(uint32_t, d[k][0]), __builtin_bit_cast(uint32_t, d[k][1]));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t y[4];   // with the low byte's carry; the low byte itself is off by 128
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = __builtin_bit_cast(uint32_t, (s2)((d[k][h] << (short)e) + (short)128));
      const uint32_t l01 = perm(y[1], y[0], 0x06020400u), l23 = perm(y[3], y[2], 0x06020400u);
      const uint32_t h01 = perm(y[1], y[0], 0x07030501u), h23 = perm(y[3], y[2], 0x07030501u);
      const int a0 = to + 4 * ((tc + 2 * h) & 15), a1 = to + 4 * ((tc + 2 * h + 1) & 15);
      sm.in.b[buf][0][a0] = perm(l23, l01, 0x05040100u) ^ 0x80808080u;
      sm.in.b[buf][0][a1] = perm(l23, l01, 0x07060302u) ^ 0x80808080u;
      sm.in.b[buf][1][a0] = perm(h23, h01, 0x05040100u);
      sm.in.b[buf][1][a1] = perm(h23, h01, 0x07060302u);
    }
  };
  // (b) co-moment sums of the raw (reference-subtracted) values
  auto comoments = [&](int buf) {
    const uint32_t* r0 = &sm.d16[buf][hy * PS + hx0 / 2 + 2];
    const uint32_t* r1 = r0 + PS;
    const uint2 x = *reinterpret_cast<const uint2*>(r0), y = *reinterpret_cast<const uint2*>(r1);
    const uint32_t x2 = r0[2], y0 = r1[-1], y3 = r1[2];
    auto lo = [&](uint32_t v) { return (float)(short)(v & 0xffffu); };
    auto hi = [&](uint32_t v) { return (float)((int)v >> 16); };
    const float a[NPX + 1] = {lo(x.x), hi(x.x), lo(x.y), hi(x.y), lo(x2)};
    const float b[NPX + 2] = {hi(y0), lo(y.x), hi(y.x), lo(y.y), hi(y.y), lo(y3)};
#pragma unroll
    for (int i = 0; i < NPX; ++i) {
      Uacc[i] += a[i];
      Pacc[0][i] = fmaf(a[i], a[i], Pacc[0][i]);
      Pacc[1][i] = fmaf(a[i], a[i + 1], Pacc[1][i]);
      Pacc[2][i] = fmaf(a[i], b[i + 1], Pacc[2][i]);
      Pacc[3][i] = fmaf(a[i], b[i + 2], Pacc[3][i]);
      Pacc[4][i] = fmaf(a[i], b[i], Pacc[4][i]);
    }
  };
  // (c) vertical pass of one block of 16 columns; lane l holds columns
  // 4 (l / 16) + 0..3 of output row l % 16
  auto vertical = [&](int blk, int buf) {
    const int g = min(q, 2);                   // rows 48 and up have no weight
    const int at = ((blk * 3 + g) * 16 + ((hy + g) & 15)) * 4;
    const i4 x0 = *reinterpret_cast<const i4*>(&sm.in.b[buf][0][at]);
    const i4 x1 = *reinterpret_cast<const i4*>(&sm.in.b[buf][1][at]);
    const i4 zero = {0, 0, 0, 0};
    // sums by their weight 2^(8 s) (of 2^30): half a unit of the result
    // starts the lowest, the byte carries (0x808080 = 131586 2^6) the
    // middle one
    i4 a0 = {1 << (29 - kFrac), 1 << (29 - kFrac), 1 << (29 - kFrac), 1 << (29 - kFrac)};
    i4 a2 = {131586, 131586, 131586, 131586};
    a0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[0], a0, 0, 0, 0);
    i4 a1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[1], zero, 0, 0, 0);
    a2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[2], a2, 0, 0, 0);
    i4 a3 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[3], zero, 0, 0, 0);
    const i4 a4 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[3], zero, 0, 0, 0);
    a1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[0], a1, 0, 0, 0);
    a2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[1], a2, 0, 0, 0);
    a3 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[2], a3, 0, 0, 0);
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int low = ((a1[i] << 8) + a0[i]) >> (30 - kFrac);
      const int top = (((a4[i] << 8) + a3[i]) << 8) + a2[i];
      v[i] = (uint32_t)((top << (kFrac - 14)) + low) ^ 0x00808080u;
    }
    const int o = blk * 64 + hy * 4 + q;
    const uint32_t p0 = perm(v[1], v[0], 0x05010400u), p1 = perm(v[3], v[2], 0x05010400u);
    const uint32_t p2 = perm(v[1], v[0], 0x07030602u), p3 = perm(v[3], v[2], 0x07030602u);
    sm.mid.b[buf][0][o] = perm(p1, p0, 0x05040100u);
    sm.mid.b[buf][1][o] = perm(p1, p0, 0x07060302u);
    sm.mid.b[buf][2][o] = perm(p3, p2, 0x05040100u);
    sm.mid.b[buf][3][o] = perm(p3, p2, 0x07060302u);
  };
  // (d) horizontal pass of this thread's pixels, in units of the lowest kept
  // product (2^16 of 2^30 weights by 2^(kFrac + e)); T and D are scaled back
  auto horizontal = [&](int buf) {
    const int at = (wv + q) * 64 + hy * 4;
    i4 x[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) x[b] = *reinterpret_cast<const i4*>(&sm.mid.b[buf][b][at]);
    i4 s[5];   // by weight 2^(8 (k + 2))
#pragma unroll
    for (int k = 0; k < 5; ++k) s[k] = i4{0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < 4; ++b)   // no product next to the one whose sum it continues
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const int o = k + 2 - b;
        if (o >= 0 && o < 4) s[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wb[b], x[o], s[k], 0, 0, 0);
      }
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double hi = (double)((s[4][i] << 8) + s[3][i]), lo = (double)((s[2][i] << 8) + s[1][i]);
      o[i] = (float)fma(fma(hi, 65536.0, lo), 256.0, (double)s[0][i]);
    }
    return make_float4(o[0], o[1], o[2], o[3]);
  };
  auto keep = [&](float (&w)[CH][NPX]) {
#pragma unroll
    for (int f = 0; f < CH; ++f) {
      const float4 v = Wl[f * NT + tid];
      w[f][0] = v.x;
      w[f][1] = v.y;
      w[f][2] = v.z;
      w[f][3] = v.w;
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < NPX; ++i) {
      Uacc[i] = 0.f;
#pragma unroll
      for (int k = 0; k < 5; ++k) Pacc[k][i] = 0.f;
    }
  };

  const double unscale = __builtin_ldexp(1.0, -(30 + kFrac - 16 + e));
  // general path: its first chunk (none yet), and the frames whose co-moments are summed
  int c0 = general ? 0 : NCH, done = 0;
  clear();
  // One barrier per frame: while frame t passes horizontally, frame t + 1
  // does vertically and frame t + 2 is staged, each in the other buffer of
  // its kind, so a wave has three independent chains.
  if (!general) {
    load(frame(0), pf);
    stage(0, 0);
    load(frame(1), pf);
    lds_barrier();
    comoments(0);
    for (int blk = wv; blk < NB; blk += 4) vertical(blk, 0);
    stage(1, 0);
    load(frame(2), pf);
    lds_barrier();
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll 1
      for (int f = 0; f < CH; ++f) {
        const int t = c * CH + f;
        const int b0 = t & 1, b1 = b0 ^ 1;
        const float4 o = horizontal(b0);
        const int first = (wv + t) & 3;   // six blocks over the four waves in turn
        if (c < NCH - 1 || t + 1 < L) {
          vertical(first, b1);
          if (first + 4 < NB) vertical(first + 4, b1);
          comoments(b1);
        }
        Wl[f * NT + tid] = o;
        if (c < NCH - 1 || t + 2 < L) {
          stage(b0, c);
          if (c < NCH - 1 || t + 3 < L) load(frame(t + 3), pf);
        }
        lds_barrier();
      }
      if (__builtin_expect(__builtin_amdgcn_readfirstlane(sm.bad[c]), 0)) {
        const bool cut = __builtin_amdgcn_readfirstlane(sm.cut) != 0;
        c0 = cut ? 0 : c;
        done = cut ? 0 : min((c + 1) * CH + 1, L);
        break;
      }
      if (c < NCH - 1) keep(win[c]);
    }
  }
  if (RARE ? __builtin_expect(c0 < NCH, 0) : __builtin_expect_with_probability(c0 < NCH, 0, 0.95)) {
    // General path, from the first chunk with a frame that does not fit: FP64
    // sums of d in FP32. The co-moments summed so far hold, unless a
    // difference may have been cut to 16 bits.
    float* Dl = sm.in.d;
    float* Ul = sm.mid.u;
    const float* own = Dl + (hy + RAD) * DW + hx0 + RAD;
    const float up = (float)__builtin_ldexp(1.0, 30 + kFrac - 16 + e);   // a power of two: values stay as rounded
    if (done == 0) clear();
    load_any(frame(c0 * CH), pf);
    lds_barrier();
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (c < c0) continue;
#pragma unroll 1
      for (int f = 0; f < CH; ++f) {
        const int t = c * CH + f;
        if (loads) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t a = pair(pf[k], sel01), b = pair(pf[k], sel23);
            const uint32_t ra = R[k][0] ^ 0x80008000u, rb = R[k][1] ^ 0x80008000u;
            *reinterpret_cast<float4*>(Dl + (4 * rq + k) * DW + 4 * cq) =
                make_float4((float)((int)(a & 0xffffu) - (int)(ra & 0xffffu)), (float)((int)(a >> 16) - (int)(ra >> 16)),
                            (float)((int)(b & 0xffffu) - (int)(rb & 0xffffu)), (float)((int)(b >> 16) - (int)(rb >> 16)));
          }
        }
        if (t + 1 < L) load_any(frame(t + 1), pf);
        lds_barrier();
        if (t >= done) {
          float a[NPX + 1], b[NPX + 2];
#pragma unroll
          for (int i = 0; i <= NPX; ++i) a[i] = own[i];
#pragma unroll
          for (int i = 0; i < NPX + 2; ++i) b[i] = own[DW - 1 + i];
#pragma unroll
          for (int i = 0; i < NPX; ++i) {
            Uacc[i] += a[i];
            Pacc[0][i] = fmaf(a[i], a[i], Pacc[0][i]);
            Pacc[1][i] = fmaf(a[i], a[i + 1], Pacc[1][i]);
            Pacc[2][i] = fmaf(a[i], b[i + 1], Pacc[2][i]);
            Pacc[3][i] = fmaf(a[i], b[i + 2], Pacc[3][i]);
            Pacc[4][i] = fmaf(a[i], b[i], Pacc[4][i]);
          }
        }
        if (tid < NVT8) vtask8(tid, Dl, Ul, p);
        lds_barrier();
        const float* row = Ul + hy * DW + hx0;
        double b0 = 0.0, b1 = 0.0, b2 = 0.0, b3 = 0.0;
#pragma unroll
        for (int j = 0; j < NTAP + 3; ++j) {
          const double x = (double)row[j];
          if (j < NTAP) b0 = fma(p.w[j], x, b0);
          if (j >= 1 && j < NTAP + 1) b1 = fma(p.w[j - 1], x, b1);
          if (j >= 2 && j < NTAP + 2) b2 = fma(p.w[j - 2], x, b2);
          if (j >= 3) b3 = fma(p.w[j - 3], x, b3);
        }
        Wl[f * NT + tid] = make_float4((float)b0 * up, (float)b1 * up, (float)b2 * up, (float)b3 * up);
      }
      if (c < NCH - 1) keep(win[c]);
    }
  }

  // ---- per-pixel selection and outputs
  const uint2 rr = *reinterpret_cast<const uint2*>(&sm.r16[hy * (TW / 2) + hx0 / 2]);
  const int gy = ty0 + hy;
#pragma unroll
  for (int i = 0; i < NPX; ++i) {
    float v[L];
#pragma unroll
    for (int s = 0; s < NCH - 1; ++s)
#pragma unroll
      for (int f = 0; f < CH; ++f) v[s * CH + f] = win[s][f][i];
#pragma unroll
    for (int f = 0; f < CH; ++f) {
      const float4 q4 = Wl[f * NT + tid];
      v[(NCH - 1) * CH + f] = i == 0 ? q4.x : i == 1 ? q4.y : i == 2 ? q4.z : q4.w;
    }
    SELNET50(v);
    const double med = 0.5 * ((double)v[SELNET50_LO] + (double)v[SELNET50_HI]);
    double lo = 0.0;
#pragma unroll
    for (int k = 0; k <= SELNET50_LO; ++k) lo += (double)v[k];
    const double dsum = (double)(L / 2) * med - lo;
    const int gx = tx0 + hx0 + i;
    if (gy < H && gx < W) {
      const long long o = (long long)(p.seg0 + sl) * M + (long long)gy * W + gx;
      const double rref = (double)((i & 1 ? (i & 2 ? rr.y : rr.x) >> 16 : (i & 2 ? rr.y : rr.x) & 0xffffu));
      p.T[o] = (float)(((double)v[SELNET50_MAX] - med) * unscale);
      p.D[o] = (float)(dsum * unscale / (double)L);
      p.S[o] = (float)(((double)L * rref + (double)Uacc[i]) / (double)L);
      p.U[o] = Uacc[i];
#pragma unroll
      for (int k = 0; k < 5; ++k) p.P[k * p.plane + o] = Pacc[k][i];
    }
  }
}

__global__ __launch_bounds__(NT, 2) void k_block_stats(KParams p) {
  __shared__ Smem sm;
  const int tiles_x = (p.W + TW - 1) / TW;
  const int tiles_y = (p.H + TH - 1) / TH;
  const int ntile = tiles_x * tiles_y;
  const int nblk = ntile * p.nseg;
  // Blocks are dealt round-robin over the 8 XCDs; give every XCD a
  // contiguous range of (segment, tile) pairs so that neighbouring tiles of a
  // segment share their halo rows in one L2.
  const int per = (nblk + 7) / 8;
  const int logical = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (logical >= nblk) return;
  const int sl = logical / ntile;
  block_body<false>(p, sl, logical - sl * ntile, sm);
}

// Serving: one persistent launch over the work items of several recordings
// described by a device-side slot table (so the launch can be captured once
// in a graph and replayed after the table is rewritten).
__global__ __launch_bounds__(NT, 2) void k_block_stats_batch(const BatchTable* __restrict__ tab) {
  __shared__ Smem sm;
  const int ns = tab->nslots;
  const int total = tab->total;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    int s = 0;
    while (s + 1 < ns && tab->slot[s + 1].item0 <= item) ++s;
    const BatchSlot& bs = tab->slot[s];
    const int local = item - bs.item0;
    const int sl = local / bs.ntile;
    const int tile = local - sl * bs.ntile;
    block_body<true>(bs.p, sl, tile, sm);
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_block_stats(const StreamLaunch& a, hipStream_t st) {
  KParams p;
  p.src0 = a.src0;
  p.src1 = a.src1;
  p.n0 = a.n0;
  p.H = a.H;
  p.W = a.W;
  p.seg0 = a.seg0;
  p.nseg = a.nseg;
  p.T = a.T;
  p.S = a.S;
  p.D = a.D;
  p.U = a.U;
  p.P = a.P;
  p.plane = a.plane;
  for (int k = 0; k < NTAP; ++k) p.w[k] = a.w[k];
  const int tiles = ((a.W + TW - 1) / TW) * ((a.H + TH - 1) / TH);
  const long long nblk = (long long)tiles * a.nseg;
  const long long per = (nblk + 7) / 8;
  hipLaunchKernelGGL(k_block_stats, dim3((unsigned)(per * 8)), dim3(NT), 0, st, p);
  return hipGetLastError();
}

size_t batch_table_bytes() { return sizeof(BatchTable); }

// Fill the host copy of the slot table; returns the number of work items.
int fill_batch_table(void* host_table, const StreamLaunch* launches, int count) {
  BatchTable* t = static_cast<BatchTable*>(host_table);
  int items = 0, ns = 0;
  for (int k = 0; k < count; ++k) {
    const StreamLaunch& a = launches[k];
    if (a.nseg <= 0) continue;
    BatchSlot& b = t->slot[ns++];
    b.p.src0 = a.src0;
    b.p.src1 = a.src1;
    b.p.n0 = a.n0;
    b.p.H = a.H;
    b.p.W = a.W;
    b.p.seg0 = a.seg0;
    b.p.nseg = a.nseg;
    b.p.T = a.T;
    b.p.S = a.S;
    b.p.D = a.D;
    b.p.U = a.U;
    b.p.P = a.P;
    b.p.plane = a.plane;
    for (int j = 0; j < NTAP; ++j) b.p.w[j] = a.w[j];
    b.ntile = ((a.W + TW - 1) / TW) * ((a.H + TH - 1) / TH);
    b.item0 = items;
    items += b.ntile * a.nseg;
  }
  t->nslots = ns;
  t->total = items;
  return items;
}

hipError_t launch_block_stats_batch(const void* dev_table, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_block_stats_batch, dim3(grid), dim3(NT), 0, st,
                     static_cast<const BatchTable*>(dev_table));
  return hipGetLastError();
}

}  // namespace seg
