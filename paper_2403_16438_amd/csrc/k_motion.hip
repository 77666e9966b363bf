// Rigid motion correction by patch-wise ZNCC (Sec. II).
//
// A frame F is compared with an integer template T: for every 21 x 21 tile
// p of F and every integer vector d with |dy|, |dx| <= R, the zero-mean
// normalised cross-correlation of F's tile with T's window at p + d. The
// per-vector sum over tiles picks the motion of the frame.
//
// With n = 441 pixels, ZNCC = (n C - sF sT) / (sqrt(vF) sqrt(vT)), where
//   C  = sum F T over the tile (the cross term),
//   sF = sum F, vF = n sum F^2 - sF^2 (per frame and tile),
//   sT = sum T, vT = n sum T^2 - sT^2 (per tile and vector, from integral
//        images of T and T^2: the table-based area sums).
// All of these are integers below 2^53, so FP64 holds them exactly; only the
// reciprocal square roots (one per frame and tile, one per tile and vector,
// from tables) and the final products round. C is a contraction of the
// template windows (rows d) with the frame tiles (columns: frames). Numerator
// and variances do not change when a constant is taken from F and from T, so
// the contraction runs on the values minus 32,896, which are exactly
// 256 hi + lo with signed bytes hi = (V >> 8) - 128 and lo = (V & 255) - 128:
// four products of bytes on the integer matrix cores, exact in INT32.
#include "seg_motion.h"

#include <mutex>

// Partial ZNCC sums of seg_mc_estimate_static, for callers that cannot
// allocate device memory: one copy per GPU, held until the process ends.
// Host code never passes this name to a kernel (on the host it is only a
// stand-in): the device address comes from mc_static_scratch below.
static __device__ __align__(256) double scratch[seg::kMcStaticDoubles];

namespace seg {
namespace {

typedef int i4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;

// ---- template -------------------------------------------------------------

// Ten frames' loads in flight per pixel: 50 frames of 256 x 256 take 5 us
// (21 us with a load per add).
__global__ void k_mc_template(const uint16_t* __restrict__ f, int n, long long M, uint16_t* __restrict__ t) {
  const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= M) return;
  uint32_t s = 0;
  int i = 0;
  for (; i + 10 <= n; i += 10) {
    uint32_t v[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) v[k] = f[(size_t)(i + k) * M + x];
#pragma unroll
    for (int k = 0; k < 10; ++k) s += v[k];
  }
  for (; i < n; ++i) s += f[(size_t)i * M + x];
  t[x] = (uint16_t)((s + (uint32_t)n / 2) / (uint32_t)n);
}

// ---- integral images and window tables --------------------------------------

// ii1, ii2: [H+1][W+1], row 0 and column 0 zero. Pass 1: running sums along
// each row, one wave per row, 64 columns per step; pass 2: down each column,
// a block of 64 columns x 16 runs of rows (each run summed, the runs' offsets
// from LDS, then its running sums). One thread per row and per column took 60
// and 79 us for 256 x 256, these 5 and 10.
__global__ __launch_bounds__(kThreads) void k_mc_rows(const uint16_t* __restrict__ t, int H, int W,
                                                      unsigned long long* __restrict__ ii1,
                                                      unsigned long long* __restrict__ ii2) {
  const int y = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (y > H) return;
  const size_t row = (size_t)y * (W + 1);
  unsigned long long a = 0, b = 0;   // sums of the columns before this step
  if (lane == 0) ii1[row] = ii2[row] = 0;
  for (int x0 = 0; x0 < W; x0 += 64) {
    const int x = x0 + lane;
    unsigned long long v = y > 0 && x < W ? t[(size_t)(y - 1) * W + x] : 0, w = v * v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long pv = __shfl_up(v, o, 64), pw = __shfl_up(w, o, 64);
      if (lane >= o) {
        v += pv;
        w += pw;
      }
    }
    v += a;
    w += b;
    if (x < W) {
      ii1[row + x + 1] = v;
      ii2[row + x + 1] = w;
    }
    a = __shfl(v, 63, 64);
    b = __shfl(w, 63, 64);
  }
}

constexpr int kColRuns = 16;
__global__ __launch_bounds__(64 * kColRuns) void k_mc_cols(int H, int W, unsigned long long* __restrict__ ii1,
                                                           unsigned long long* __restrict__ ii2) {
  __shared__ unsigned long long s[kColRuns][64];
  const int lane = threadIdx.x & 63, run = threadIdx.x >> 6, x = blockIdx.x * 64 + lane;
  const int len = (H + kColRuns) / kColRuns, y0 = run * len, y1 = min(H + 1, y0 + len);   // H + 1 rows
  unsigned long long* ii = blockIdx.y ? ii2 : ii1;
  unsigned long long a = 0;
  if (x <= W)
#pragma unroll 8
    for (int y = y0; y < y1; ++y) a += ii[(size_t)y * (W + 1) + x];
  s[run][lane] = a;
  __syncthreads();
  a = 0;
  for (int r = 0; r < run; ++r) a += s[r][lane];
  if (x > W) return;
  for (int y = y0; y < y1; y += 8) {
    unsigned long long v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = ii[(size_t)min(y + k, y1 - 1) * (W + 1) + x];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (y + k < y1) {
        a += v[k];
        ii[(size_t)(y + k) * (W + 1) + x] = a;
      }
  }
}

__global__ void k_mc_windows(McGeom g, const unsigned long long* __restrict__ ii1,
                             const unsigned long long* __restrict__ ii2, double* sT, double* vT) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.P * g.Vp) return;
  const int p = i / g.Vp, v = i % g.Vp;
  if (v >= g.V) {
    sT[i] = 0.0;
    vT[i] = 0.0;
    return;
  }
  const int side = 2 * g.R + 1;
  const int y0 = g.oy + (p / g.nx) * kPatch + v / side - g.R;
  const int x0 = g.ox + (p % g.nx) * kPatch + v % side - g.R;
  const size_t w1 = (size_t)g.W + 1;
  auto box = [&](const unsigned long long* ii) {
    return ii[(size_t)(y0 + kPatch) * w1 + x0 + kPatch] - ii[(size_t)y0 * w1 + x0 + kPatch] -
           ii[(size_t)(y0 + kPatch) * w1 + x0] + ii[(size_t)y0 * w1 + x0];
  };
  const long long s1 = (long long)box(ii1), s2 = (long long)box(ii2);
  const long long var = kPatchPix * s2 - s1 * s1;
  sT[i] = (double)s1;
  vT[i] = var > 0 ? 1.0 / sqrt((double)var) : 0.0;   // 0: zero variance, ZNCC 0
}

// ---- scores -------------------------------------------------------------------

// Depth layout of a tile's 441 pixels, 512 bytes: 32 groups of 16 bytes, four
// groups per MFMA step. Groups 0..19 are columns 0..15 of rows 0..19; group
// 20 + h (h = 0..10) holds columns 16..23 of rows 2 h and 2 h + 1; group 31
// holds columns 0..15 of row 20. Columns past 20 and row 21 are zero on the
// frame's side, so what the template's side reads there does not count.
constexpr int kSteps = 8;
constexpr int kFS = 528;                 // bytes of one frame's tile in LDS (512 and a 16-byte shift of the banks)
// The template window lies in LDS four times, shifted by 0..3 bytes, so that
// the 16 columns that a vector (dy, dx) wants start at a whole 32-bit word of
// copy dx % 4. Rows of 16 words and copies 676 words apart (36 modulo the 64
// banks) put the 64 words that a wave reads at once (four rows, four copies,
// four words) on 64 banks.
constexpr int kTR = 16, kTC = 676;
constexpr int kMaxTW = kPatch + 2 * kMcMaxRadius;
constexpr int kMaxVp = ((2 * kMcMaxRadius + 1) * (2 * kMcMaxRadius + 1) + 15) / 16 * 16;
static_assert((kMaxTW + 1) * kTR <= kTC, "a copy holds the window and the row below it");
constexpr int kOff = 32896;              // 256 * 128 + 128
constexpr int kSFrames = 16;             // frames per workgroup (the MFMA's columns)
constexpr int kNV = 3;                   // vector tiles that a wave takes at a time

struct ScoreLds {
  uint32_t th[4 * kTC], tl[4 * kTC];     // template window, high and low bytes
  uint8_t fh[kSFrames * kFS], fl[kSFrames * kFS];
  double sT[kMaxVp], vT[kMaxVp];
  double sf[kSFrames], rf[kSFrames];       // moments of the frames' tiles
};

__device__ __forceinline__ uint32_t lo4(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x06040200u); }
__device__ __forceinline__ uint32_t hi4(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07050301u); }

// What a thread loads of the next tile while the present one is computed: 8
// pixels of up to three rows of the template window, some rows of one frame's
// tile, and entries of the window tables.
struct Prefetch {
  static constexpr int G = kThreads / kSFrames;        // threads per frame
  static constexpr int NR = (kPatch + G - 1) / G;       // rows per thread
  static constexpr int TR = (kMaxTW + 15) / 16;
  uint32_t t[TR][4], d[NR][11];
  double st[2], vt[2];
};

// Template window of tile (py, px): thread (row pass, j) takes pixels 4 j ..
// 4 j + 7 of a row and writes word j of the four copies. Frame tiles: thread
// (f, sub) takes every G-th row of frame f's tile, 21 pixels at any 2-byte
// address, as 11 aligned words.
__device__ __forceinline__ void load_tile(Prefetch& pf, const McScoreArgs& a, const uint16_t* __restrict__ frames,
                                          long long M, int nf, int p, int v0, int v1) {
  const McGeom& g = a.g;
  const int py = g.oy + (p / g.nx) * kPatch, px = g.ox + (p % g.nx) * kPatch;
  const int f = threadIdx.x / pf.G, sub = threadIdx.x % pf.G;
  const uint16_t* src = frames + (size_t)min(f, nf - 1) * M + (size_t)py * g.W + px;
#pragma unroll
  for (int k = 0; k < pf.NR; ++k) {
    const uint16_t* row = src + (size_t)min(sub + pf.G * k, kPatch - 1) * g.W;
    row -= (uintptr_t)row >> 1 & 1;
    __builtin_memcpy(pf.d[k], __builtin_assume_aligned(row, 4), 44);
  }
  const int j = min((int)(threadIdx.x & 15), g.R / 2 + 5);
#pragma unroll
  for (int k = 0; k < pf.TR; ++k) {
    const int r = min((int)(threadIdx.x >> 4) + 16 * k, g.TW - 1);
    __builtin_memcpy(pf.t[k], a.tmpl + (size_t)(py - g.R + r) * g.W + (px - g.R + 4 * j), 16);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int d = min(v0 * 16 + (int)threadIdx.x + kThreads * k, v1 * 16 - 1);
    pf.st[k] = a.sT[(size_t)p * g.Vp + d];
    pf.vt[k] = a.vT[(size_t)p * g.Vp + d];
  }
}

// The loaded tile into LDS.
__device__ __forceinline__ void store_tile(ScoreLds& sm, const Prefetch& pf, const McScoreArgs& a,
                                           const uint16_t* __restrict__ frames, long long M, int nf, int p, int v0,
                                           int v1) {
  const McGeom& g = a.g;
  const int py = g.oy + (p / g.nx) * kPatch, px = g.ox + (p % g.nx) * kPatch;
  const int j = threadIdx.x & 15;
  if (j < g.R / 2 + 6) {   // words that dx = 2 R reaches
#pragma unroll
    for (int k = 0; k < pf.TR; ++k) {
      const int at = min((int)(threadIdx.x >> 4) + 16 * k, g.TW - 1) * kTR + j;
      const uint32_t* w = pf.t[k];
      const uint32_t l0 = lo4(w[0], w[1]) ^ 0x80808080u, l1 = lo4(w[2], w[3]) ^ 0x80808080u;
      const uint32_t h0 = hi4(w[0], w[1]) ^ 0x80808080u, h1 = hi4(w[2], w[3]) ^ 0x80808080u;
      sm.tl[at] = l0;
      sm.th[at] = h0;
#pragma unroll
      for (int c = 1; c < 4; ++c) {
        sm.tl[c * kTC + at] = __builtin_amdgcn_alignbit(l1, l0, 8 * c);
        sm.th[c * kTC + at] = __builtin_amdgcn_alignbit(h1, h0, 8 * c);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int d = v0 * 16 + (int)threadIdx.x + kThreads * k;
    if (d < v1 * 16) {
      sm.sT[d] = pf.st[k] - (double)(kPatchPix * kOff);
      sm.vT[d] = pf.vt[k];
    }
  }
  const int f = threadIdx.x / pf.G, sub = threadIdx.x % pf.G;
  const uint16_t* src = frames + (size_t)min(f, nf - 1) * M + (size_t)py * g.W + px;
#pragma unroll
  for (int k = 0; k < pf.NR; ++k) {
    const int r = sub + pf.G * k;
    if (r >= kPatch) break;
    const int odd = (int)((uintptr_t)(src + (size_t)r * g.W) >> 1 & 1);
    uint32_t w[11];
#pragma unroll
    for (int i = 0; i < 10; ++i) w[i] = __builtin_amdgcn_alignbit(pf.d[k][i + 1], pf.d[k][i], 16 * odd);
    w[10] = pf.d[k][10] >> 16 * odd;
    uint32_t l[6], h[6];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      l[i] = lo4(w[2 * i], w[2 * i + 1]) ^ 0x80808080u;
      h[i] = hi4(w[2 * i], w[2 * i + 1]) ^ 0x80808080u;
    }
    l[5] = (w[10] & 0xffu) ^ 0x80u;
    h[5] = (w[10] >> 8 & 0xffu) ^ 0x80u;
    if (f >= nf) {
#pragma unroll
      for (int i = 0; i < 6; ++i) l[i] = h[i] = 0;
    }
    const int at = f * kFS + (r < 20 ? r : 31) * 16, b = f * kFS + (20 + (r >> 1)) * 16 + (r & 1) * 8;
    *reinterpret_cast<uint4*>(&sm.fl[at]) = make_uint4(l[0], l[1], l[2], l[3]);
    *reinterpret_cast<uint4*>(&sm.fh[at]) = make_uint4(h[0], h[1], h[2], h[3]);
    *reinterpret_cast<uint2*>(&sm.fl[b]) = make_uint2(l[4], l[5]);
    *reinterpret_cast<uint2*>(&sm.fh[b]) = make_uint2(h[4], h[5]);
    if (r == 20) {
      *reinterpret_cast<uint2*>(&sm.fl[b + 8]) = make_uint2(0, 0);
      *reinterpret_cast<uint2*>(&sm.fh[b + 8]) = make_uint2(0, 0);
    }
  }
}

// Moments of the 16 frames' tile, by one wave: the products of the frames with
// themselves (sums of squares on the diagonal) and with ones.
__device__ __forceinline__ void tile_moments(ScoreLds& sm, int lane) {
  const int q = lane >> 4, col = lane & 15, at = col * kFS + q * 16;
  const i4 one = {0x01010101, 0x01010101, 0x01010101, 0x01010101}, z = {0, 0, 0, 0};
  i4 hh = z, hl = z, ll = z, sh = z, sl = z;
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const i4 bh = *reinterpret_cast<const i4*>(&sm.fh[at + 64 * s]);
    const i4 bl = *reinterpret_cast<const i4*>(&sm.fl[at + 64 * s]);
    hh = __builtin_amdgcn_mfma_i32_16x16x64_i8(bh, bh, hh, 0, 0, 0);
    hl = __builtin_amdgcn_mfma_i32_16x16x64_i8(bh, bl, hl, 0, 0, 0);
    ll = __builtin_amdgcn_mfma_i32_16x16x64_i8(bl, bl, ll, 0, 0, 0);
    sh = __builtin_amdgcn_mfma_i32_16x16x64_i8(one, bh, sh, 0, 0, 0);
    sl = __builtin_amdgcn_mfma_i32_16x16x64_i8(one, bl, sl, 0, 0, 0);
  }
  if (col >> 2 != q) return;   // row 4 q + col % 4 = column col
  const int i = col & 3;
  auto pick = [i](const i4& v) { return i == 0 ? v[0] : i == 1 ? v[1] : i == 2 ? v[2] : v[3]; };
  const int s = 256 * sh[0] + sl[0];
  const long long v = kPatchPix * (65536LL * pick(hh) + 512LL * pick(hl) + pick(ll)) - (long long)s * s;
  sm.sf[col] = (double)s;
  sm.rf[col] = v > 0 ? 1.0 / sqrt((double)v) : 0.0;
}

// The cross terms of NV vector tiles (template words base[i0 + i] for this
// lane's vector) with the frames' tile: high by high bytes, the two mixed
// products, low by low.
template <int NV, int TPW>
__device__ __forceinline__ void cross_terms(i4 (&hh)[kNV], i4 (&x)[kNV], i4 (&ll)[kNV], const ScoreLds& sm,
                                            const int (&base)[TPW], int i0, int lane) {
  const int q = lane >> 4, at = (lane & 15) * kFS + q * 16;
#pragma unroll
  for (int i = 0; i < NV; ++i) hh[i] = x[i] = ll[i] = i4{0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const i4 bh = *reinterpret_cast<const i4*>(&sm.fh[at + 64 * s]);
    const i4 bl = *reinterpret_cast<const i4*>(&sm.fl[at + 64 * s]);
    i4 ah[NV], al[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int b = base[i0 + i];
      int a0, a1;   // words of the group's first and second half
      if (s < 5) {
        a0 = b + (4 * s + q) * kTR;
        a1 = a0 + 2;
      } else {
        a0 = b + 2 * (4 * (s - 5) + q) * kTR + 4;
        a1 = a0 + kTR;
        if (s == 7 && q == 3) {
          a0 = b + 20 * kTR;
          a1 = a0 + 2;
        }
      }
      ah[i] = i4{(int)sm.th[a0], (int)sm.th[a0 + 1], (int)sm.th[a1], (int)sm.th[a1 + 1]};
      al[i] = i4{(int)sm.tl[a0], (int)sm.tl[a0 + 1], (int)sm.tl[a1], (int)sm.tl[a1 + 1]};
    }
    // no product next to the one whose sum it continues
#pragma unroll
    for (int i = 0; i < NV; ++i) x[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah[i], bl, x[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NV; ++i) hh[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah[i], bh, hh[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NV; ++i) x[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[i], bh, x[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NV; ++i) ll[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al[i], bl, ll[i], 0, 0, 0);
  }
}

// One workgroup: 16 frames, one slice of tiles, and the vector tiles v0 ..
// v1 - 1, of which wave w owns v0 + w, v0 + w + 4, ... (at most TPW). INT8
// MFMA 16x16x64: lane l supplies row (column) l % 16 of A (B) with the depth
// group 4 step + l / 16, and holds rows 4 (l / 16) + 0..3 of column l % 16;
// rows are vectors, columns frames.
//
// 2,000 frames of 256 x 256 at radius 8: 280 us, where the same sums on
// v_mfma_f64_16x16x4f64 took 1,598 us; 50 frames of 128 x 128: 14 us and 122.
// By leaving parts out: the cross terms take 128 us of it (their operands'
// LDS reads; the matrix cores need 61), the epilogue 16, and staging the next
// tile 77, half of that its writes to LDS. Two tiles by 32 frames per operand,
// or two or three neighbouring tiles staged at once, needed more registers
// than two workgroups per compute unit have and took 275 to 420 us.
template <int TPW>
__global__ __launch_bounds__(kThreads, 2) void k_mc_scores(McScoreArgs a, int VG, int per) {
  __shared__ __attribute__((aligned(16))) ScoreLds sm;
  const McGeom g = a.g;
  const int vg = blockIdx.x % VG, slice = blockIdx.x / VG % g.S, grp = blockIdx.x / VG / g.S;
  const int f0 = grp * kSFrames, nf = min(kSFrames, a.n - f0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, q = lane >> 4;
  const int side = 2 * g.R + 1;
  const int v0 = vg * per, v1 = min(v0 + per, g.Vp / 16);
  const int nt = min(TPW, max(0, (v1 - v0 - wave + 3) / 4));   // vector tiles of this wave
  const long long M = (long long)g.H * g.W;
  const uint16_t* frames = a.frames + (size_t)f0 * M;

  int base[TPW];
  double score[TPW][4];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int d = (v0 + wave + 4 * i) * 16 + col;
    const int dy = d / side, dx = d - dy * side;
    base[i] = (i < nt && d < g.V) ? (dx & 3) * kTC + dy * kTR + (dx >> 2) : 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) score[i][r] = 0.0;
  }

  const int p0 = slice * g.pps, p1 = min(g.P, p0 + g.pps);
  Prefetch pf;
  load_tile(pf, a, frames, M, nf, p0, v0, v1);
  for (int p = p0; p < p1; ++p) {
    __syncthreads();
    store_tile(sm, pf, a, frames, M, nf, p, v0, v1);
    __syncthreads();
    if (p + 1 < p1) load_tile(pf, a, frames, M, nf, p + 1, v0, v1);
    if (wave == 3) tile_moments(sm, lane);   // the wave with the fewest vector tiles
#pragma unroll
    for (int i0 = 0; i0 < TPW; i0 += kNV) {   // the count of vector tiles is wave-uniform
      i4 hh[kNV], x[kNV], ll[kNV];
      const int n = min(nt - i0, kNV);
      if (TPW - i0 >= 3 && n == 3)
        cross_terms<3>(hh, x, ll, sm, base, i0, lane);
      else if (TPW - i0 >= 2 && n == 2)
        cross_terms<2>(hh, x, ll, sm, base, i0, lane);
      else if (n == 1)
        cross_terms<1>(hh, x, ll, sm, base, i0, lane);
      if (i0 == 0) __syncthreads();   // the moments are there
      const double sf = sm.sf[col], rf = sm.rf[col];
#pragma unroll
      for (int i = 0; i < kNV; ++i) {
        if (i0 + i >= TPW || i >= n) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int d = (v0 + wave + 4 * (i0 + i)) * 16 + 4 * q + r;
          // |256 hh + x| < 2^31: 441 products of bytes each
          const double c = fma((double)(hh[i][r] * 256 + x[i][r]), 256.0, (double)ll[i][r]);
          score[i0 + i][r] += ((double)kPatchPix * c - sf * sm.sT[d]) * rf * sm.vT[d];
        }
      }
    }
  }
  if (col >= nf) return;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (i >= nt) break;
    const int d = (v0 + wave + 4 * i) * 16 + 4 * q;
    double* out = a.part + ((size_t)slice * a.chunk + f0 + col) * g.Vp + d;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = score[i][r];
  }
}

// ---- pick and apply -----------------------------------------------------------

// One wave per frame: lanes take vectors d = lane, lane + 64, ...; the slice
// sums are added in slice order; the first maximum wins.
__global__ __launch_bounds__(kThreads) void k_mc_pick(McGeom g, const double* __restrict__ part, int chunk,
                                                      int n, int32_t* motion, double* scores) {
  const int f = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (f >= n) return;
  double best = -1.0e300;
  int arg = 0x7fffffff;
  for (int d = lane; d < g.V; d += 64) {
    double v[kMcSlices], s = 0.0;   // all slices' loads in flight
#pragma unroll
    for (int sl = 0; sl < kMcSlices; ++sl) v[sl] = part[((size_t)min(sl, g.S - 1) * chunk + f) * g.Vp + d];
#pragma unroll
    for (int sl = 0; sl < kMcSlices; ++sl)
      if (sl < g.S) s += v[sl];
    if (scores) scores[(size_t)f * g.V + d] = s;
    if (s > best) {
      best = s;
      arg = d;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    if (ob > best || (ob == best && oa < arg)) {
      best = ob;
      arg = oa;
    }
  }
  if (lane == 0) {
    const int side = 2 * g.R + 1;
    motion[2 * (size_t)f] = -(arg / side - g.R);
    motion[2 * (size_t)f + 1] = -(arg % side - g.R);
  }
}

// C(y, x) = F(y + my, x + mx) where that pixel is in the frame, else the
// template's T(y, x). Grid: x runs over the 8-pixel runs of a frame, y over
// frames (uniform motion per workgroup); each thread gathers one run and
// writes it with one 16-byte store. Frame widths that are not a multiple of
// 8 take the per-pixel kernel.
__global__ void k_mc_apply8(const uint16_t* __restrict__ in, int H, int W, const int32_t* __restrict__ motion,
                            const uint16_t* __restrict__ tmpl, uint16_t* __restrict__ out) {
  const int runs = W >> 3;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= H * runs) return;
  const size_t f = blockIdx.y;
  const int y = i / runs, x0 = (i - y * runs) << 3;
  const int my = motion[2 * f], mx = motion[2 * f + 1];
  const size_t M = (size_t)H * W;
  const int sy = y + my;
  const uint16_t* trow = tmpl + (size_t)y * W + x0;
  uint16_t v[8];
  if (sy < 0 || sy >= H) {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = trow[k];
  } else {
    const uint16_t* srow = in + f * M + (size_t)sy * W;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int sx = x0 + k + mx;
      v[k] = (sx >= 0 && sx < W) ? srow[sx] : trow[k];
    }
  }
  uint4 pk;
  pk.x = v[0] | ((uint32_t)v[1] << 16);
  pk.y = v[2] | ((uint32_t)v[3] << 16);
  pk.z = v[4] | ((uint32_t)v[5] << 16);
  pk.w = v[6] | ((uint32_t)v[7] << 16);
  *reinterpret_cast<uint4*>(out + f * M + (size_t)y * W + x0) = pk;
}

__global__ void k_mc_apply1(const uint16_t* __restrict__ in, int H, int W, const int32_t* __restrict__ motion,
                            const uint16_t* __restrict__ tmpl, uint16_t* __restrict__ out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= H * W) return;
  const size_t f = blockIdx.y, M = (size_t)H * W;
  const int y = r / W, x = r % W;
  const int sy = y + motion[2 * f], sx = x + motion[2 * f + 1];
  const bool inside = sy >= 0 && sy < H && sx >= 0 && sx < W;
  out[f * M + r] = inside ? in[f * M + (size_t)sy * W + sx] : tmpl[r];
}

}  // namespace

hipError_t launch_mc_template(const uint16_t* frames, int n, long long M, uint16_t* tmpl, hipStream_t st) {
  hipLaunchKernelGGL(k_mc_template, dim3((unsigned)((M + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                     frames, n, M, tmpl);
  return hipGetLastError();
}

hipError_t launch_mc_tables(const McGeom& g, const uint16_t* tmpl, unsigned long long* ii, double* sT,
                            double* vT, hipStream_t st) {
  unsigned long long* ii2 = ii + (size_t)(g.H + 1) * (g.W + 1);
  hipLaunchKernelGGL(k_mc_rows, dim3((g.H + 1 + kThreads / 64 - 1) / (kThreads / 64)), dim3(kThreads), 0, st, tmpl, g.H, g.W, ii, ii2);
  hipLaunchKernelGGL(k_mc_cols, dim3((g.W + 1 + 63) / 64, 2), dim3(64 * kColRuns), 0, st, g.H, g.W, ii, ii2);
  const int n = g.P * g.Vp;
  hipLaunchKernelGGL(k_mc_windows, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, st, g, ii, ii2, sT,
                     vT);
  return hipGetLastError();
}

// The split never changes a score: a vector's sum over the tiles of a slice
// is formed in one place, whatever vectors share its workgroup. A workgroup
// takes up to 20 vector tiles (five per wave), so that few read the same
// frames; with fewer frames than fill the chip (two workgroups per compute
// unit) the vectors are dealt to more workgroups, down to one tile per wave.
hipError_t launch_mc_scores(const McScoreArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  const int MT = a.g.Vp / 16, units = (a.n + kSFrames - 1) / kSFrames * a.g.S;
  int VG = (MT + 19) / 20;
  while (units * VG < 512 && VG < (MT + 3) / 4) ++VG;
  const int per = (MT + VG - 1) / VG;
  VG = (MT + per - 1) / per;
  const dim3 grid((unsigned)(units * VG)), block(kThreads);
  switch ((per + 3) / 4) {
    case 1: hipLaunchKernelGGL(k_mc_scores<1>, grid, block, 0, st, a, VG, per); break;
    case 2: hipLaunchKernelGGL(k_mc_scores<2>, grid, block, 0, st, a, VG, per); break;
    case 3: hipLaunchKernelGGL(k_mc_scores<3>, grid, block, 0, st, a, VG, per); break;
    case 4: hipLaunchKernelGGL(k_mc_scores<4>, grid, block, 0, st, a, VG, per); break;
    case 5: hipLaunchKernelGGL(k_mc_scores<5>, grid, block, 0, st, a, VG, per); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_mc_pick(const McGeom& g, const double* part, int chunk, int n, int32_t* motion,
                          double* scores, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int per = kThreads / 64;
  hipLaunchKernelGGL(k_mc_pick, dim3((unsigned)((n + per - 1) / per)), dim3(kThreads), 0, st, g, part, chunk, n,
                     motion, scores);
  return hipGetLastError();
}

hipError_t launch_mc_apply(const uint16_t* in, long long n, int H, int W, const int32_t* motion,
                           const uint16_t* tmpl, uint16_t* out, hipStream_t st) {
  const bool vec = W % 8 == 0 && ((uintptr_t)out & 15) == 0;
  const long long per = vec ? (long long)H * (W / 8) : (long long)H * W;
  const unsigned bx = (unsigned)((per + kThreads - 1) / kThreads);
  for (long long f0 = 0; f0 < n; f0 += 65535) {
    const unsigned nf = (unsigned)(n - f0 < 65535 ? n - f0 : 65535);
    const size_t o = (size_t)f0 * H * W;
    if (vec)
      hipLaunchKernelGGL(k_mc_apply8, dim3(bx, nf), dim3(kThreads), 0, st, in + o, H, W, motion + 2 * f0, tmpl,
                         out + o);
    else
      hipLaunchKernelGGL(k_mc_apply1, dim3(bx, nf), dim3(kThreads), 0, st, in + o, H, W, motion + 2 * f0, tmpl,
                         out + o);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t mc_static_scratch(double** ptr) {
  static std::mutex mu;
  static double* cache[kMaxMcDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxMcDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> hold(mu);
  if (!cache[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    cache[dev] = static_cast<double*>(p);
  }
  *ptr = cache[dev];
  return hipSuccess;
}

}  // namespace seg
