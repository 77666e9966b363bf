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
// runs on INT8 MFMA in fixed point: d is two signed bytes and a weight (a whole
// number of 2^-30 to 2^-32) four, so the vertical pass is eight byte products,
// exact in INT32; its result, rounded to 28 + e fraction bits, is five bytes,
// and the horizontal pass leaves out the three of twenty byte products that are
// below 2^-40 of the range. One FP64 sum per value restores it, exact but for
// that rounding, and rounds it to FP32. The scale e is the tile's, 0 to 3, with
// |d| 2^e at most 2,000 (four times the range of the first three frames where
// that fits); a frame past it takes e = -4 for itself, |d| up to 32,000.
//
// Accuracy: a smoothed value has one rounding to 2^-(28 + e) and one to FP32,
// where FP64 sums with an FP32 intermediate have two to FP32. The first is the
// smaller error in T from T = 0.1 sqrt(sum w^2) 2^-e on, e the smallest of the
// segment's frames (0.03 at sigma 3 and e = 0: noise of sd 0.14). A segment of a tile with a fainter pixel among those
// whose own values vary, one with |d| above 32,000 and frames narrower than four
// pixels take the general path: FP64 sums over 25 taps in both passes. (A pixel
// that is constant itself and sees others' noise at the kernel's edge keeps the
// absolute error.) Mean relative error of T against FP64, here and of FP64 sums
// with an FP32 intermediate: noise of sd 33 3.0e-8 and 3.4e-8; of sd 10, 3 and 1
// beside 4 x 4 pixels of sd 400, 400 and 450 3.1e-8, 3.0e-8 and 3.0e-8 and
// 3.4e-8 each. Four bytes of 20 + e fraction bits, e up to 7, had 3.6e-8, 5.6e-8
// and 1.1e-7 there, and single pixels beyond 2e-6.
//
// What bounds it: vector instructions of the two waves that a SIMD holds (the
// FP32 window, 200 values of a thread, allows no third), then the chain from
// staging through both passes where a launch has one workgroup per compute
// unit. Hence 16-bit arithmetic while staging, byte planes laid out as the
// matrix operands read them, and one barrier per frame with the three steps
// of three frames between two. Measured, from FP64 sums and two barriers per
// frame (which also read a width that is no multiple of four pixel by pixel):
// 64 x 64 x 50 99 -> 81 us, 450 x 138 x 500 561 -> 172 us, four recordings of
// 500 frames in one launch (128 x 128 to 512 x 512) 1,515 -> 934 us (the four
// bytes above: 80, 168 and 1,000 us). 256 x 256 x 1,600: 586 -> 449 us, with
// bright frames in every segment 573 -> 438 us, and with values over the whole
// 16-bit range, which take the general path, 578 -> 577 us (138 x 450 x 500 490
// -> 220 us).
//
// Every thread owns 4 adjacent pixels of one tile row and keeps their 50
// smoothed values in VGPRs (40) and a per-thread LDS slot (the chunk being
// filled); after the segment a compare-exchange network gives the median, the
// maximum and the 25 smallest values.
#include <cmath>

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
  int seg0;
  float quiet;   // T from which the fixed point is as exact as FP32 at scale 0
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

// General path: vertical pass for one (column, 8-row) task: U rows 8h..8h+7 of column c,
// streaming the 32 staged rows once.
constexpr int VROWS = 8;
constexpr int NVT8 = DW * (TH / VROWS);   // 176 tasks, one round
constexpr int UW = DW + 4;                // words per row of U: 16 rows' 16-byte reads on all banks
static_assert(NVT8 <= NT, "one vertical round");

__device__ __forceinline__ void vtask8(int q, const float* __restrict__ Dl,
                                       float* __restrict__ Ul, const double (&w)[NTAP]) {
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
      if (j - o >= 0 && j - o < NTAP) acc[o] = fma(w[j - o], x, acc[o]);
  }
  float* out = Ul + h * VROWS * UW + c;
#pragma unroll
  for (int o = 0; o < VROWS; ++o) out[o * UW] = (float)acc[o];
}

typedef int i4 __attribute__((ext_vector_type(4)));
typedef short s2 __attribute__((ext_vector_type(2)));
typedef unsigned short u2 __attribute__((ext_vector_type(2)));
typedef uint32_t px4 __attribute__((ext_vector_type(2), aligned(2)));   // four pixels at any pixel's address
typedef const __attribute__((address_space(1))) uint16_t* gpixels;
typedef const __attribute__((address_space(1))) char* gbytes;
typedef __attribute__((address_space(1))) float* gfloats;

// Staging: thread cq 10 + rq takes the 4 x 4 pixels of rows 4 rq .. and
// columns 4 cq .. of the staged region, so that the bytes of four rows of a
// column are one LDS word. One 8-byte load and a byte permutation fetch four
// columns.
constexpr int QR = DH / 4, QC = DW / 4;   // 10 x 22 items
static_assert(QR * QC <= NT, "one item per thread");
constexpr int NB = 6;                     // blocks of 16 staged columns (the last one half used)
constexpr int PR = TH + 4;                // staged rows 12 .. 31 ..
constexpr int PS = TW / 2 + 4;            // .. and columns 8 .. 79 as 16-bit pairs: words per row
constexpr int MB = 5;                     // bytes of the intermediate
// A frame's scale e: |d| 2^e at most kRange, so that the upper four bytes of
// the intermediate (20 + e fraction bits of 28 + e) and their carries are below
// 2^31.
constexpr int kRange = 2000, kFrac = 28;
constexpr int kLoud = -4, kLoudRange = kRange << -kLoud;   // the scale of a frame past its tile's

struct Smem {
  union {
    struct {
      // Operands lie as the lanes of a wave read them, 16 bytes each in a row:
      // [block][16 rows][column] low and high bytes of d, and [block][row] the
      // bytes of 16 columns of the intermediate, lowest byte first. Even and
      // odd frames have their own.
      uint32_t in[2][2][NB * 3 * 16 * 4];
      uint32_t mid[2][MB][NB * 16 * 4];
      uint32_t d16[2][PR * PS];
    } x;
    uint32_t r16[TH * TW / 2];     // at the end: R of the tile's own pixels
    struct {                       // general path: d, R and the intermediate
      float d[DH * DW], r[DH * DW], u[TH * UW];
    } g;
  };
  float4 Wl[CH * NT];
  int loud[L];                 // frames past the tile's scale
  int leave[NCH + 1];          // the general path is wanted: a frame staged in this chunk, a faint pixel
  int top[4];
};
static_assert(sizeof(Smem) <= 80 * 1024, "two workgroups per compute unit");

__device__ __forceinline__ int med3i(int a, int b, int c) { return max(min(a, b), min(max(a, b), c)); }

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}

// 16 output values from 40 inputs along the depth of a 16 x 16 x 64 product:
// lane l holds, for output l % 16, the four bytes (lowest first) of the
// weights of inputs 16 (l / 16) .. + 15: w[input - output] times `scale`.
__device__ __forceinline__ void band(const __attribute__((address_space(4))) double* w, double scale, int lane, i4 (&wb)[4]) {
  const int m = lane & 15, k0 = 16 * (lane >> 4);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int tap = k0 + 4 * j + u - m;
      const double x = tap >= 0 && tap < NTAP ? w[min(max(tap, 0), NTAP - 1)] : 0.0;
      // signed bytes: a byte above 127 is taken off and carried to the next
      q[u] = ((uint32_t)(int)__builtin_rint(x * scale) + 0x00808080u) ^ 0x00808080u;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t sel = 0x0c0c0000u | (uint32_t)(4 + b) << 8 | (uint32_t)b;   // byte b of both, zeros above
      wb[b][j] = (int)perm(perm(q[3], q[2], sel), perm(q[1], q[0], sel), 0x05040100u);
    }
  }
}

typedef __attribute__((address_space(3))) Smem* LdsSmem;
typedef const __attribute__((address_space(4))) KParams* ConstParams;

// Global memory by its address space: pointers that come from the slot table
// would be accessed with generic instructions, which an LDS barrier waits for.
struct Frames {
  const uint16_t *src0, *src1;
  long long n0, first, M;
  __device__ __forceinline__ gpixels operator()(int t) const {
    const long long f = first + t;
    return (gpixels)(f < n0 ? src0 + f * M : src1 + (f - n0) * M);
  }
};
__device__ __forceinline__ Frames frames_of(ConstParams p, int sl) {
  return {p->src0, p->src1, p->n0, (long long)sl * L, (long long)p->H * p->W};
}

struct Out {
  gfloats T, S, D, U, P;
  long long plane;
  int H, W, seg0;
};
__device__ __forceinline__ Out outputs(ConstParams p) {
  return {(gfloats)p->T, (gfloats)p->S, (gfloats)p->D, (gfloats)p->U, (gfloats)p->P, p->plane, p->H, p->W, p->seg0};
}

// Four neighbouring columns, folded at the frame's border in whatever way, lie
// in four contiguous source columns: the first of these, and the bytes of
// columns 0, 1 and 2, 3 among the eight.
__device__ __forceinline__ int columns(int x, int W, uint32_t& sel01, uint32_t& sel23) {
  int c[4], lo = W;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    c[i] = reflect(x + i, W);
    lo = min(lo, c[i]);
  }
  lo = max(min(lo, W - 4), 0);
  auto bytes = [&](int i) { return (uint32_t)(2 * (c[i] - lo)) * 0x0101u + 0x0100u; };
  sel01 = bytes(0) | bytes(1) << 16;
  sel23 = bytes(2) | bytes(3) << 16;
  return lo;
}
__device__ __forceinline__ uint2 load_columns(gpixels fr, unsigned off) {
  const px4 w = *(const __attribute__((address_space(1))) px4*)((gbytes)fr + off);
  return make_uint2(w.x, w.y);
}
// the same where a row has fewer than four pixels, read one by one
__device__ __forceinline__ uint2 load_narrow(gpixels fr, unsigned off, int W) {
  const gpixels r = (gpixels)((gbytes)fr + off);
  return make_uint2((uint32_t)r[0] | (uint32_t)r[min(1, W - 1)] << 16, r[min(2, W - 1)]);
}

// the chunk in a thread's LDS slots into its registers
__device__ __forceinline__ void keep(const float4* Wl, float (&w)[CH][NPX]) {
#pragma unroll
  for (int f = 0; f < CH; ++f) {
    const float4 v = Wl[f * NT];
    w[f][0] = v.x;
    w[f][1] = v.y;
    w[f][2] = v.z;
    w[f][3] = v.w;
  }
}

// The segment's maps and co-moment sums of a thread's four pixels from their
// window: chunks 0 .. 3 in registers, the last one in its LDS slots. Says whether
// a pixel whose own value varies has a T below `quiet`.
__device__ __forceinline__ bool store_pixels(const Out& p, int sl, int gy, int gx0, const float (&win)[NCH - 1][CH][NPX],
                                             const float4* Wl, const float (&Uacc)[NPX], const float (&Pacc)[5][NPX],
                                             const float (&rref)[NPX], double unit, float quiet) {
  bool faint = false;
#pragma unroll
  for (int i = 0; i < NPX; ++i) {
    float v[L];
#pragma unroll
    for (int s = 0; s < NCH - 1; ++s)
#pragma unroll
      for (int f = 0; f < CH; ++f) v[s * CH + f] = win[s][f][i];
#pragma unroll
    for (int f = 0; f < CH; ++f) {
      const float4 q4 = Wl[f * NT];
      v[(NCH - 1) * CH + f] = i == 0 ? q4.x : i == 1 ? q4.y : i == 2 ? q4.z : q4.w;
    }
    SELNET50(v);
    const double med = 0.5 * ((double)v[SELNET50_LO] + (double)v[SELNET50_HI]);
    double lo = 0.0;
#pragma unroll
    for (int k = 0; k <= SELNET50_LO; ++k) lo += (double)v[k];
    const double dsum = (double)(L / 2) * med - lo;
    const int gx = gx0 + i;
    if (gy < p.H && gx < p.W) {
      const long long o = (long long)(p.seg0 + sl) * p.H * p.W + (long long)gy * p.W + gx;
      const float T = (float)(((double)v[SELNET50_MAX] - med) * unit);
      faint |= Pacc[0][i] > 0.f && T < quiet;
      p.T[o] = T;
      p.D[o] = (float)(dsum * unit / (double)L);
      p.S[o] = (float)(((double)L * (double)rref[i] + (double)Uacc[i]) / (double)L);
      p.U[o] = Uacc[i];
#pragma unroll
      for (int k = 0; k < 5; ++k) p.P[k * p.plane + o] = Pacc[k][i];
    }
  }
  return faint;
}

// The general path: FP64 sums of d in FP32, from the segment's first frame, so
// that no register lives on from the fixed-point path: with its window and
// scale handed over in one body, frames that all come here took 660 us at
// 256 x 256 x 1,600 (now 577). NARROW: rows of fewer than four pixels.
template <bool NARROW>
__device__ __forceinline__ void general_segment(ConstParams p, int sl, int tile, Smem& sm) {
  const Out out = outputs(p);
  const int H = out.H, W = out.W;
  double w[NTAP];
#pragma unroll
  for (int k = 0; k < NTAP; ++k) w[k] = p->w[k];
  float* Dl = sm.g.d;
  float* Rl = sm.g.r;
  float* Ul = sm.g.u;
  float4* Wl = sm.Wl;
  const int tid = threadIdx.x, lane = tid & 63;
  const int tiles_x = (W + TW - 1) / TW;
  const int ty0 = (tile / tiles_x) * TH, tx0 = (tile % tiles_x) * TW;
  const int hy = lane & 15, hx0 = 16 * __builtin_amdgcn_readfirstlane(tid >> 6) + 4 * (lane >> 4);
  const Frames frame = frames_of(p, sl);

  // staging: 40 rows of 22 groups of four columns, up to four groups per thread
  constexpr int NQ = DH * QC, KQ = (NQ + NT - 1) / NT;
  unsigned off[KQ];
  uint32_t sel01[KQ], sel23[KQ];
#pragma unroll
  for (int k = 0; k < KQ; ++k) {
    const int g = min(tid + k * NT, NQ - 1), r = g / QC;
    const int lo = columns(tx0 - RAD + 4 * (g - r * QC), W, sel01[k], sel23[k]);
    off[k] = 2u * (unsigned)(reflect(ty0 - RAD + r, H) * W + lo);
  }
  const int nk = tid + (KQ - 1) * NT < NQ ? KQ : KQ - 1;
  auto load = [&](int t, uint2 (&v)[KQ]) {
    const gpixels fr = frame(t);
#pragma unroll
    for (int k = 0; k < KQ; ++k) v[k] = NARROW ? load_narrow(fr, off[k], W) : load_columns(fr, off[k]);
  };
  auto pixels = [&](uint2 v, int k) {
    const uint32_t a = perm(v.y, v.x, sel01[k]), b = perm(v.y, v.x, sel23[k]);
    return make_int4((int)(a & 0xffffu), (int)(a >> 16), (int)(b & 0xffffu), (int)(b >> 16));
  };
  __syncthreads();   // the fixed-point path's reads of the same LDS
  uint2 pf[KQ];
  {
    uint2 f1[KQ], f2[KQ];
    load(0, pf);
    load(1, f1);
    load(2, f2);
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
      const int4 a = pixels(pf[k], k), b = pixels(f1[k], k), c = pixels(f2[k], k);
      if (k < nk)
        *reinterpret_cast<float4*>(Rl + 4 * (tid + k * NT)) = make_float4(
            (float)med3i(a.x, b.x, c.x), (float)med3i(a.y, b.y, c.y), (float)med3i(a.z, b.z, c.z), (float)med3i(a.w, b.w, c.w));
    }
  }

  float win[NCH - 1][CH][NPX], Uacc[NPX], Pacc[5][NPX];
#pragma unroll
  for (int i = 0; i < NPX; ++i) {
    Uacc[i] = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) Pacc[k][i] = 0.f;
  }
  const float* own = Dl + (hy + RAD) * DW + hx0 + RAD;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
#pragma unroll 1
    for (int f = 0; f < CH; ++f) {
      const int t = c * CH + f;
      // (a) stage d = V - R for the tile and its halo
#pragma unroll
      for (int k = 0; k < KQ; ++k)
        if (k < nk) {
          const int4 x = pixels(pf[k], k);
          const float4 r = *reinterpret_cast<const float4*>(Rl + 4 * (tid + k * NT));
          *reinterpret_cast<float4*>(Dl + 4 * (tid + k * NT)) =
              make_float4((float)x.x - r.x, (float)x.y - r.y, (float)x.z - r.z, (float)x.w - r.w);
        }
      if (t + 1 < L) load(t + 1, pf);
      lds_barrier();
      // (b) co-moment sums of the raw (reference-subtracted) values
      {
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
      // (c) vertical pass
      if (tid < NVT8) vtask8(tid, Dl, Ul, w);
      lds_barrier();
      // (d) horizontal pass into this thread's LDS chunk slot
      const float* row = Ul + hy * UW + hx0;
      double b0 = 0.0, b1 = 0.0, b2 = 0.0, b3 = 0.0;
#pragma unroll
      for (int j = 0; j < NTAP + 3; ++j) {
        const double x = (double)row[j];
        if (j < NTAP) b0 = fma(w[j], x, b0);
        if (j >= 1 && j < NTAP + 1) b1 = fma(w[j - 1], x, b1);
        if (j >= 2 && j < NTAP + 2) b2 = fma(w[j - 2], x, b2);
        if (j >= 3) b3 = fma(w[j - 3], x, b3);
      }
      Wl[f * NT + tid] = make_float4((float)b0, (float)b1, (float)b2, (float)b3);
    }
    if (c < NCH - 1) keep(Wl + tid, win[c]);
  }
  float rref[NPX];
#pragma unroll
  for (int i = 0; i < NPX; ++i) rref[i] = Rl[(hy + RAD) * DW + hx0 + RAD + i];
  store_pixels(out, sl, ty0 + hy, tx0 + hx0, win, Wl + tid, Uacc, Pacc, rref, 1.0, 0.f);
}

// One (segment sl, tile) work item of one recording in fixed point; false if
// it is one for the general path.
template <bool BATCH>
__device__ __forceinline__ bool fixed_segment(ConstParams params, int sl, int tile, Smem& sm) {
  float4* Wl = sm.Wl;
  int tid = threadIdx.x;
  // what follows from the thread's number is formed anew for each item rather
  // than kept in scratch around the batch kernel's loop
  if constexpr (BATCH) asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Out out = outputs(params);
  const int W = out.W, H = out.H;
  if (W < 4) return false;
  const int tiles_x = (W + TW - 1) / TW;
  const int ty0 = (tile / tiles_x) * TH;
  const int tx0 = (tile % tiles_x) * TW;
  const Frames frame = frames_of(params, sl);

  // ---- staging geometry
  const bool loads = tid < QR * QC;
  const int cq = loads ? tid / QR : 0, rq = loads ? tid - cq * QR : 0;
  unsigned off[4];         // byte offset of the first of the four source columns, per row
  uint32_t sel01, sel23;   // bytes of columns 0, 1 and 2, 3 among the eight loaded
  {
    const int lo = columns(tx0 - RAD + 4 * cq, W, sel01, sel23);
#pragma unroll
    for (int k = 0; k < 4; ++k) off[k] = 2u * (unsigned)(reflect(ty0 - RAD + 4 * rq + k, H) * W + lo);
  }
  // four rows of four pixels, as loaded
  auto load = [&](gpixels fr, uint2 (&v)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = load_columns(fr, off[k]);
  };
  auto pair = [&](uint2 v, uint32_t sel) { return perm(v.y, v.x, sel); };
  const bool centre = loads && rq >= RAD / 4 && rq < (RAD + PR) / 4 && cq >= 2 && cq < 2 + PS / 2;

  // ---- per-pixel reference: median of the segment's first three frames, and
  // the tile's scale from the largest |V - R| among them
  // the weights as whole numbers of 2^-wbits: the largest and its byte carries
  // are below 2^31
  const double most = params->w[RAD];
  const int wbits = __builtin_amdgcn_readfirstlane(most > 0.99 ? 30 : most > 0.49 ? 31 : 32);
  uint32_t R[4][2];
  int e;
  {
    uint2 f0[4], f1[4], f2[4];
    load(frame(0), f0);
    load(frame(1), f1);
    load(frame(2), f2);
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
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      R[k][0] ^= 0x80008000u;   // as the signed subtraction below wants it
      R[k][1] ^= 0x80008000u;
    }
    int t = max((int)top.x, (int)top.y);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t = max(t, __shfl_xor(t, o, 64));
    if (lane == 0) sm.top[wv] = t;
    if (tid < L) sm.loud[tid] = 0;
    if (tid <= NCH) sm.leave[tid] = 0;
    __syncthreads();
    t = __builtin_amdgcn_readfirstlane(max(max(max(sm.top[0], sm.top[1]), max(sm.top[2], sm.top[3])), 1));
    if (t > kLoudRange) return false;
    e = 0;
    while (e < wbits - kFrac - 1 && 4 * t << (e + 1) <= kRange) ++e;
  }
  const short lim = (short)(kRange >> e);

  // ---- thread-owned pixels: tile row hy, columns hx0 .. hx0+3 (the layout of
  // the horizontal product's result)
  const int hy = lane & 15, q = lane >> 4;
  const int hx0 = 16 * wv + 4 * q;

  i4 wb[4];
  band(params->w, __builtin_ldexp(1.0, wbits), lane, wb);

  // 40 of the 50 window values live in VGPRs (chunks 0..3); the chunk being
  // filled lives in a per-thread LDS slot, so the frame loop needs no
  // compile-time frame index. The chunk loop is unrolled, so a completed
  // chunk c moves once into its own registers win[c].
  float win[NCH - 1][CH][NPX];
  // Co-moment sums: U is exact, P while 50 d^2 is below 2^24 (|d| up to 579).
  float Uacc[NPX], Pacc[5][NPX];

  // (a) stage d = V - R of the tile and its halo from the prefetched frame
  uint2 pf[4];
  const int to = (((cq >> 2) * 3 + (rq >> 2)) * 16) * 4 + (rq & 3);
  const int tc = 4 * (cq & 3) + (rq >> 2);   // columns turned by the row block: fewer lanes on one bank
  auto stage = [&](int buf, int t, int c) {
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
    if (max((int)over.x, (int)over.y) > 2 * lim) {
      sm.loud[t] = 1;
      bool cut = false;
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          cut |= max(abs((int)d[k][h].x), abs((int)d[k][h].y)) > kLoudRange;
      if (cut) sm.leave[c] = 1;
    }
    if (centre) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<uint2*>(&sm.x.d16[buf][(4 * rq + k - RAD) * PS + 2 * cq - 4]) =
            make_uint2(__builtin_bit_cast(uint32_t, d[k][0]), __builtin_bit_cast(uint32_t, d[k][1]));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t y[4];   // with the low byte's carry; the low byte itself is off by 128
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = __builtin_bit_cast(uint32_t, (s2)(d[k][h] + (short)128));
      const uint32_t l01 = perm(y[1], y[0], 0x06020400u), l23 = perm(y[3], y[2], 0x06020400u);
      const uint32_t h01 = perm(y[1], y[0], 0x07030501u), h23 = perm(y[3], y[2], 0x07030501u);
      const int a0 = to + 4 * ((tc + 2 * h) & 15), a1 = to + 4 * ((tc + 2 * h + 1) & 15);
      sm.x.in[buf][0][a0] = perm(l23, l01, 0x05040100u) ^ 0x80808080u;
      sm.x.in[buf][0][a1] = perm(l23, l01, 0x07060302u) ^ 0x80808080u;
      sm.x.in[buf][1][a0] = perm(h23, h01, 0x05040100u);
      sm.x.in[buf][1][a1] = perm(h23, h01, 0x07060302u);
    }
  };
  // (b) co-moment sums of the raw (reference-subtracted) values
  auto comoments = [&](int buf) {
    const uint32_t* r0 = &sm.x.d16[buf][hy * PS + hx0 / 2 + 2];
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
  // (c) vertical pass of one block of 16 columns of a frame of scale x; lane l
  // holds columns 4 (l / 16) + 0..3 of output row l % 16
  auto vertical = [&](int blk, int buf, int x) {
    const int g = min(q, 2);                   // rows 48 and up have no weight
    const int at = ((blk * 3 + g) * 16 + ((hy + g) & 15)) * 4;
    const i4 x0 = *reinterpret_cast<const i4*>(&sm.x.in[buf][0][at]);
    const i4 x1 = *reinterpret_cast<const i4*>(&sm.x.in[buf][1][at]);
    const i4 zero = {0, 0, 0, 0};
    // sums by their weight 2^(8 s - wbits); `low` bits of them are below the
    // result (1 to 8). The lowest starts with half a unit of the result and the
    // carry of its lowest byte, the middle one with the other bytes' carries.
    const int low = wbits - kFrac - x;
    const int c0 = (1 << (low - 1)) + (128 << low), c2 = 0x00808080 >> (8 - low);
    i4 a0 = {c0, c0, c0, c0}, a2 = {c2, c2, c2, c2};
    a0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[0], a0, 0, 0, 0);
    i4 a1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[1], zero, 0, 0, 0);
    a2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[2], a2, 0, 0, 0);
    i4 a3 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, wb[3], zero, 0, 0, 0);
    const i4 a4 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[3], zero, 0, 0, 0);
    a1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[0], a1, 0, 0, 0);
    a2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[1], a2, 0, 0, 0);
    a3 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, wb[2], a3, 0, 0, 0);
    uint32_t u[4], v[4];   // the lowest byte, and the other four
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = ((a1[i] << 8) + a0[i]) >> low;
      const uint32_t t = ((((uint32_t)a4[i] << 8) + (uint32_t)a3[i]) << 8) + (uint32_t)a2[i];
      u[i] = (uint32_t)b;
      v[i] = ((t << (8 - low)) + (uint32_t)(b >> 8)) ^ 0x00808080u;
    }
    const int o = blk * 64 + hy * 4 + q;
    const uint32_t p0 = perm(v[1], v[0], 0x05010400u), p1 = perm(v[3], v[2], 0x05010400u);
    const uint32_t p2 = perm(v[1], v[0], 0x07030602u), p3 = perm(v[3], v[2], 0x07030602u);
    sm.x.mid[buf][0][o] = perm(perm(u[3], u[2], 0x0c0c0400u), perm(u[1], u[0], 0x0c0c0400u), 0x05040100u) ^ 0x80808080u;
    sm.x.mid[buf][1][o] = perm(p1, p0, 0x05040100u);
    sm.x.mid[buf][2][o] = perm(p1, p0, 0x07060302u);
    sm.x.mid[buf][3][o] = perm(p3, p2, 0x05040100u);
    sm.x.mid[buf][4][o] = perm(p3, p2, 0x07060302u);
  };
  // (d) horizontal pass of this thread's pixels of a frame of scale x
  auto horizontal = [&](int buf, int x) {
    // the last group's last block of columns has no weight
    const int at = min(wv + q, NB - 1) * 64 + hy * 4;
    i4 y[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) y[b] = *reinterpret_cast<const i4*>(&sm.x.mid[buf][b][at]);
    i4 s[6];   // by weight 2^(8 (k + 2))
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] = i4{0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < MB; ++b)   // no product next to the one whose sum it continues
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int o = k + 2 - b;
        if (o >= 0 && o < 4) s[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wb[o], y[b], s[k], 0, 0, 0);
      }
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double hi = (double)((s[5][i] << 8) + s[4][i]), mid = (double)((s[3][i] << 8) + s[2][i]),
                   lo = (double)((s[1][i] << 8) + s[0][i]);
      o[i] = (float)fma(fma(hi, 65536.0, mid), 65536.0, lo);
    }
    if (x != e) {   // in units of the tile's scale
      const float by = __builtin_ldexpf(1.f, e - x);
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] *= by;
    }
    return make_float4(o[0], o[1], o[2], o[3]);
  };
  auto scale = [&](int t) { return __builtin_amdgcn_readfirstlane(sm.loud[t]) ? kLoud : e; };

#pragma unroll
  for (int i = 0; i < NPX; ++i) {
    Uacc[i] = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) Pacc[k][i] = 0.f;
  }
  // One barrier per frame: while frame t passes horizontally, frame t + 1
  // does vertically and frame t + 2 is staged, each in the other buffer of
  // its kind, so a wave has three independent chains.
  load(frame(0), pf);
  stage(0, 0, 0);
  load(frame(1), pf);
  lds_barrier();
  int x0 = scale(0), least = x0;   // scale of frame t, and the smallest
  comoments(0);
  for (int blk = wv; blk < NB; blk += 4) vertical(blk, 0, x0);
  stage(1, 1, 0);
  load(frame(2), pf);
  lds_barrier();
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
#pragma unroll 1
    for (int f = 0; f < CH; ++f) {
      const int t = c * CH + f;
      const int b0 = t & 1, b1 = b0 ^ 1;
      const int x1 = scale(min(t + 1, L - 1));
      const float4 o = horizontal(b0, x0);
      const int first = (wv + t) & 3;   // six blocks over the four waves in turn
      if (c < NCH - 1 || t + 1 < L) {
        vertical(first, b1, x1);
        if (first + 4 < NB) vertical(first + 4, b1, x1);
        comoments(b1);
      }
      Wl[f * NT + tid] = o;
      if (c < NCH - 1 || t + 2 < L) {
        stage(b0, t + 2, c);
        if (c < NCH - 1 || t + 3 < L) load(frame(t + 3), pf);
      }
      x0 = x1;
      least = min(least, x1);
      lds_barrier();
    }
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(sm.leave[c]), 0)) return false;
    if (c < NCH - 1) keep(Wl + tid, win[c]);
  }

  // ---- R to the pixels' owners, selection and outputs
  if (loads && rq >= RAD / 4 && rq < (RAD + TH) / 4 && cq >= RAD / 4 && cq < (RAD + TW) / 4) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *reinterpret_cast<uint2*>(&sm.r16[(4 * rq + k - RAD) * (TW / 2) + 2 * cq - RAD / 2]) =
          make_uint2(R[k][0] ^ 0x80008000u, R[k][1] ^ 0x80008000u);
  }
  lds_barrier();
  const uint2 rr = *reinterpret_cast<const uint2*>(&sm.r16[hy * (TW / 2) + hx0 / 2]);
  const float rref[NPX] = {(float)(rr.x & 0xffffu), (float)(rr.x >> 16), (float)(rr.y & 0xffffu), (float)(rr.y >> 16)};
  const float quiet = params->quiet * __builtin_ldexpf(1.f, -least);
  if (store_pixels(out, sl, ty0 + hy, tx0 + hx0, win, Wl + tid, Uacc, Pacc, rref,
                   __builtin_ldexp(1.0, 16 - kFrac - wbits - e), quiet))
    sm.leave[NCH] = 1;
  __syncthreads();
  return !__builtin_amdgcn_readfirstlane(sm.leave[NCH]);
}

// The general path called: its arguments come in vector registers, and the
// compiler is to know that the LDS is aligned (four-byte LDS reads otherwise:
// 625 -> 655 us). The batch kernel, short of registers for its loop over items,
// and narrow frames call it; a call saves 112 registers per thread, and where
// all segments take it costs 25 us more.
template <bool NARROW>
__device__ __attribute__((noinline)) void general_call(ConstParams params, int sl, int tile, LdsSmem lds) {
  const uint64_t p = (uint64_t)params;
  const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)lds) & ~15u;
  general_segment<NARROW>((ConstParams)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) << 32 |
                                        (uint32_t)__builtin_amdgcn_readfirstlane((int)p)),
                          __builtin_amdgcn_readfirstlane(sl), __builtin_amdgcn_readfirstlane(tile),
                          *(Smem*)(LdsSmem)(uintptr_t)at);
}

template <bool BATCH>
__device__ __forceinline__ void work_item(ConstParams params, int sl, int tile, Smem& sm) {
  if (fixed_segment<BATCH>(params, sl, tile, sm)) return;
  if (params->W < 4) general_call<true>(params, sl, tile, (LdsSmem)&sm);
  else if (BATCH) general_call<false>(params, sl, tile, (LdsSmem)&sm);
  else general_segment<false>(params, sl, tile, sm);
}

__global__ __launch_bounds__(NT, 2) void k_block_stats(KParams p, int nseg) {
  __shared__ Smem sm;
  const int tiles_x = (p.W + TW - 1) / TW;
  const int tiles_y = (p.H + TH - 1) / TH;
  const int ntile = tiles_x * tiles_y;
  const int nblk = ntile * nseg;
  // Blocks are dealt round-robin over the 8 XCDs; give every XCD a
  // contiguous range of (segment, tile) pairs so that neighbouring tiles of a
  // segment share their halo rows in one L2.
  const int per = (nblk + 7) / 8;
  const int logical = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (logical >= nblk) return;
  const int sl = logical / ntile;
  work_item<false>((ConstParams)__builtin_amdgcn_kernarg_segment_ptr(), sl, logical - sl * ntile, sm);
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
    work_item<true>((ConstParams)&bs.p, sl, tile, sm);
    __syncthreads();
  }
}

}  // namespace

namespace {
KParams params_of(const StreamLaunch& a) {
  KParams p;
  p.src0 = a.src0;
  p.src1 = a.src1;
  p.n0 = a.n0;
  p.H = a.H;
  p.W = a.W;
  p.seg0 = a.seg0;
  p.T = a.T;
  p.S = a.S;
  p.D = a.D;
  p.U = a.U;
  p.P = a.P;
  p.plane = a.plane;
  double gain = 0.0;
  for (int k = 0; k < NTAP; ++k) {
    p.w[k] = a.w[k];
    gain += a.w[k] * a.w[k];
  }
  p.quiet = (float)(0.1 * std::sqrt(gain));
  return p;
}
}  // namespace

hipError_t launch_block_stats(const StreamLaunch& a, hipStream_t st) {
  const KParams p = params_of(a);
  const int tiles = ((a.W + TW - 1) / TW) * ((a.H + TH - 1) / TH);
  const long long nblk = (long long)tiles * a.nseg;
  const long long per = (nblk + 7) / 8;
  hipLaunchKernelGGL(k_block_stats, dim3((unsigned)(per * 8)), dim3(NT), 0, st, p, a.nseg);
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
    b.p = params_of(a);
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
