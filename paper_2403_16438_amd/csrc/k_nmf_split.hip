// Per-component NMF P_c ~ F A (Eq. 3, Sec. III-D) with each component split
// over several workgroups that run at the same time (cooperative launch).
//
// Workgroup w of component c owns a contiguous range of the component's
// pixels (rows of P_c) and keeps those rows of P_c in LDS (FP32, exact) for
// the whole factorisation, with an odd row stride so that both the row-wise
// and the column-wise sweeps are free of bank conflicts. Everything that needs
// all pixels of the component is a sum (or max) over pixels, so each
// workgroup writes its partial over its own rows to an exchange slot in HBM,
// and each workgroup of the component waits for and adds the slots of all of
// them in the same fixed order. They thus hold bit-identical
// totals and take identical decisions without further communication:
//   SPA     per step: partial squared column norms of the residual, then the
//           partial projections onto the picked direction (two exchanges);
//           the residual rows stay with their owner (HBM, owner-only)
//   init    partial maxima of the picked columns (one exchange)
//   HALS    per sweep one exchange of the partial F^T F and F^T P; every
//           workgroup then runs the same A update (A is small and is kept
//           whole in each workgroup's LDS), forms A A^T itself and updates
//           the F rows it owns from its LDS rows of P_c
//   scale   partial column maxima of F (one exchange)
// The arithmetic is the single-workgroup kernel's (same update order, FP64,
// clipping, zero-Gram rule); only the summation order of the sums differs.
// A sweep has five workgroup barriers: after the F^T P partials, after the
// gather, after the A update, after the P A^T partials and after the F
// update; the Gram matrices are formed within one wave, which needs none.
//
// Exchange: every slot value travels as two 64-bit words (its high and low
// halves), each tagged in its upper 32 bits with the number of the exchange
// that wrote it, and written and read with relaxed agent-scope atomics. A
// word read with the expected tag therefore holds that exchange's half
// (single-copy atomicity of the word), so readers poll the slot words
// themselves: no arrival counter, no fences, and the values are exact. Two
// slots per workgroup alternate between exchanges; a workgroup can only
// overwrite a slot after every workgroup of its component has read it (it
// needs their next slots first), and the slots are cleared before each
// launch, so a stale word never carries the expected tag. The launch is
// cooperative (unless every component is one workgroup's: nothing is exchanged
// then), so all workgroups are resident; a wait is still bounded by a
// wall-clock limit, after which the component is marked abandoned, every
// workgroup of it leaves, and the error flag is set.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "seg_kernels.h"

namespace seg {
namespace {

constexpr int R8 = kMaxRank;

__device__ __forceinline__ double wsum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// pair k of the upper triangle of an NR x NR matrix, row by row
template <int NR>
__device__ __forceinline__ void pair_of(int k, int& n1, int& n2) {
  n1 = 0;
  while (k >= NR - n1) {
    k -= NR - n1;
    ++n1;
  }
  n2 = n1 + k;
}

// X^T X of the first NR columns of X [len][R8] (LDS) by the 64 lanes of one
// wave: lane (chunk q, entry p of the upper triangle) sums its chunk of rows
// for entry p, the QG chunk partials go to part [QG][NP] (LDS), and lane p < NP
// adds the partials of entry p in chunk order. Returns that total in lanes
// p < NP (0 elsewhere). The wave needs no barrier: the LDS requests of a wave
// complete in order.
template <int NR>
__device__ __forceinline__ double gram_wave(const double* X, int len, int lane, double* part) {
  constexpr int NP = NR * (NR + 1) / 2;
  constexpr int QG = NP <= 4 ? 16 : NP <= 8 ? 8 : NP <= 16 ? 4 : NP <= 32 ? 2 : 1;
  if (lane < QG * NP) {
    const int q = lane / NP, p = lane - q * NP;
    int n1, n2;
    pair_of<NR>(p, n1, n2);
    const int span = (len + QG - 1) / QG, j1 = min(len, (q + 1) * span);
    double g0 = 0.0, g1 = 0.0;
    int j = q * span;
    for (; j + 3 < j1; j += 4) {
      double x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        x[u] = X[(j + u) * R8 + n1];
        y[u] = X[(j + u) * R8 + n2];
      }
      g0 = fma(x[0], y[0], g0);
      g1 = fma(x[1], y[1], g1);
      g0 = fma(x[2], y[2], g0);
      g1 = fma(x[3], y[3], g1);
    }
    for (; j + 1 < j1; j += 2) {
      g0 = fma(X[j * R8 + n1], X[j * R8 + n2], g0);
      g1 = fma(X[(j + 1) * R8 + n1], X[(j + 1) * R8 + n2], g1);
    }
    if (j < j1) g0 = fma(X[j * R8 + n1], X[j * R8 + n2], g0);
    part[q * NP + p] = g0 + g1;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  double v = 0.0;
  if (lane < NP) {
    double x[QG];
#pragma unroll
    for (int q = 0; q < QG; ++q) x[q] = part[q * NP + lane];
    v = x[0];
#pragma unroll
    for (int q = 1; q < QG; ++q) v += x[q];
  }
  return v;
}

// in-order sum x[0] + x[step] + ... + x[(n - 1) step], n <= 16, loads issued
// in groups of four ahead of the adds
__device__ __forceinline__ double chunk_sum(const double* x, size_t step, int n) {
  double v = x[0];
  int q = 1;
  for (; q + 3 < n; q += 4) {
    const double a = x[q * step], b = x[(q + 1) * step], c = x[(q + 2) * step], d = x[(q + 3) * step];
    v += a;
    v += b;
    v += c;
    v += d;
  }
  for (; q < n; ++q) v += x[q * step];
  return v;
}

template <int CW>
__device__ double block_max(double v, double* red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  if (lane == 0) red[w] = v;
  __syncthreads();
  double m = red[0];
  for (int ww = 1; ww < CW; ++ww) m = fmax(m, red[ww]);
  __syncthreads();
  return m;
}

// argmax with lowest index on ties
template <int CW>
__device__ void block_argmax(double v, int idx, double* red, int* redi, double* best, int* bidx) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(v, off);
    const int oi = __shfl_xor(idx, off);
    if (ov > v || (ov == v && oi < idx)) {
      v = ov;
      idx = oi;
    }
  }
  if (lane == 0) {
    red[w] = v;
    redi[w] = idx;
  }
  __syncthreads();
  double b = red[0];
  int bi = redi[0];
  for (int ww = 1; ww < CW; ++ww)
    if (red[ww] > b || (red[ww] == b && redi[ww] < bi)) {
      b = red[ww];
      bi = redi[ww];
    }
  *best = b;
  *bidx = bi;
  __syncthreads();
}

using u64 = unsigned long long;

// ---- short components: HALS with the rows of P_c in registers
//
// A component that one workgroup holds whole, of at most 512 pixels, 44
// segments and rank 3: a thread of the first four waves keeps its one or two
// rows of P_c and of F in registers, a lane its column of A, and a sweep has one
// barrier. F^T P and F^T F are summed over a wave's rows by halving exchanges,
// sixteen sums at a time (eight values against eight with the other half of the
// wave, then four, two, one), over the waves through LDS; every wave then forms
// the same A and takes its columns as scalars for the rows of P A^T. What
// bounds it is the instructions of one wave per SIMD, the divisions' chains
// among them. The NMF of a 64 x 64 x 1,000 recording (three components of 200
// to 300 pixels, rank 1, 200 sweeps) takes 0.32 ms; with P_c in LDS, five
// barriers a sweep and an exchange of slots between two workgroups it took
// 0.90. At rank 2 and 370 pixels 0.75 against 1.14 ms (all eight waves with one
// row each: 1.00; 1,024 threads and so half the registers: 1.07). A component
// whose rank turns out to be higher (the plan is made before the projections
// find it) is left, marked by kNmfLeft in place of its rank, for the launch
// that splits components.
constexpr int kRowsMax = 512, kRowsK = 44, kRowsRank = 3;

__device__ __forceinline__ double swap_add32(double a, double b) {
  const u64 x = (u64)__double_as_longlong(a), y = (u64)__double_as_longlong(b);
  const auto l = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return __longlong_as_double((long long)((u64)h[0] << 32 | l[0])) + __longlong_as_double((long long)((u64)h[1] << 32 | l[1]));
}

__device__ __forceinline__ double swap_add16(double a, double b) {
  const u64 x = (u64)__double_as_longlong(a), y = (u64)__double_as_longlong(b);
  const auto l = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return __longlong_as_double((long long)((u64)h[0] << 32 | l[0])) + __longlong_as_double((long long)((u64)h[1] << 32 | l[1]));
}

template <int CTRL>
__device__ __forceinline__ double from_lane(double v) {
  const u64 x = (u64)__double_as_longlong(v);
  const int l = __builtin_amdgcn_update_dpp(0, (int)(unsigned)x, CTRL, 0xf, 0xf, false);
  const int h = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)((u64)(unsigned)h << 32 | (unsigned)l));
}

// sum of v[i] over the wave's lanes, in lanes 4 i .. 4 i + 3
__device__ __forceinline__ double wave_sums(double (&v)[16], int lane) {
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = swap_add32(v[i], v[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = swap_add16(v[i], v[i + 4]);
  const bool b3 = lane & 8, b2 = lane & 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) v[i] = (b3 ? v[i + 2] : v[i]) + from_lane<0x128>(b3 ? v[i] : v[i + 2]);   // row_ror 8
  double x = (b2 ? v[1] : v[0]) + from_lane<0x141>(b2 ? v[0] : v[1]);   // row_half_mirror: the other quad
  x += from_lane<0x4e>(x);   // quad_perm 2, 3, 0, 1
  x += from_lane<0xb1>(x);   // quad_perm 1, 0, 3, 2
  return x;
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const u64 x = (u64)__double_as_longlong(v);
  const unsigned l = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, lane);
  const unsigned h = (unsigned)__builtin_amdgcn_readlane((int)(x >> 32), lane);
  return __longlong_as_double((long long)((u64)h << 32 | l));
}

// doubles of LDS: two sets of the waves' sums
constexpr int rows_scratch(int K) { return 2 * 4 * kRowsRank * ((K + kRowsRank + 15) / 16 * 16); }

// RP rows per thread of the first four waves, NR rank, KC blocks of 16
// columns: K columns of P_c, and in the last NR the entries (n, n2) of F^T F,
// n2 >= n
template <int RP, int NR, int KC>
__device__ void hals_rows(const float* Pl, int Kp, double* F, double* A, double* part, int ml, int K, int sweeps) {
  constexpr int KW = 16 * KC, G0 = KW - NR;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, nwv = min(4, (ml + 63) >> 6);
  const bool col = lane < K;
  float p[RP][KW];
  double f[RP][NR], av[NR];
  bool row[RP];
#pragma unroll
  for (int u = 0; u < RP; ++u) {
    const int m = t + 256 * u;
    row[u] = t < 256 && m < ml;
#pragma unroll
    for (int i = 0; i < KW; ++i) p[u][i] = row[u] && i < K ? Pl[m * Kp + i] : 0.f;
#pragma unroll
    for (int n = 0; n < NR; ++n) f[u][n] = row[u] ? F[m * R8 + n] : 0.0;
  }
#pragma unroll
  for (int n = 0; n < NR; ++n) av[n] = 0.0;
  for (int sweep = -1; sweep < sweeps; ++sweep) {
    double* set = part + (sweep & 1) * nwv * NR * KW;
    if (wv < nwv) {
#pragma unroll
      for (int n = 0; n < NR; ++n)
#pragma unroll
        for (int c = 0; c < KC; ++c) {
          double v[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int k = 16 * c + i, n2 = k - G0;
            if (n2 >= 0 && n2 < n) {   // (n2, n) is row n2's
              v[i] = 0.0;
              continue;
            }
#pragma unroll
            for (int u = 0; u < RP; ++u) {
              const double y = n2 >= 0 ? f[u][n2 < 0 ? 0 : n2] : (double)p[u][k];
              v[i] = u == 0 ? f[u][n] * y : fma(f[u][n], y, v[i]);
            }
          }
          const double x = wave_sums(v, lane);
          if ((lane & 3) == 0) set[(wv * NR + n) * KW + 16 * c + (lane >> 2)] = x;
        }
    }
    __syncthreads();
    if (wv >= nwv) continue;
    double tot[NR], g[NR][NR];
#pragma unroll
    for (int n = 0; n < NR; ++n) {
      const double* x = set + n * KW + min(lane, KW - 1);
      tot[n] = x[0];
      for (int w = 1; w < nwv; ++w) tot[n] += x[w * NR * KW];
    }
#pragma unroll
    for (int n = 0; n < NR; ++n)
#pragma unroll
      for (int n2 = n; n2 < NR; ++n2) g[n][n2] = g[n2][n] = lane_value(tot[n], G0 + n2);
#pragma unroll
    for (int n = 0; n < NR; ++n)
      if (g[n][n] > 0.0) {
        double sg = 0.0;
#pragma unroll
        for (int n2 = 0; n2 < NR; ++n2) sg += g[n][n2] * av[n2];
        av[n] = col ? fmax(0.0, av[n] + (tot[n] - sg) / g[n][n]) : 0.0;
      }
    if (sweep < 0) continue;
    // A A^T over the lanes, P A^T over the columns of A as scalars
    double aa[NR][NR];
    {
      double v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = 0.0;
#pragma unroll
      for (int n = 0, i = 0; n < NR; ++n)
#pragma unroll
        for (int n2 = n; n2 < NR; ++n2, ++i) v[i] = av[n] * av[n2];
      const double x = wave_sums(v, lane);
#pragma unroll
      for (int n = 0, i = 0; n < NR; ++n)
#pragma unroll
        for (int n2 = n; n2 < NR; ++n2, ++i) aa[n][n2] = aa[n2][n] = lane_value(x, 4 * i);
    }
    double gp[RP][NR][2];
#pragma unroll
    for (int u = 0; u < RP; ++u)
#pragma unroll
      for (int n = 0; n < NR; ++n) gp[u][n][0] = gp[u][n][1] = 0.0;
#pragma unroll
    for (int k = 0; k < G0; ++k) {
#pragma unroll
      for (int n = 0; n < NR; ++n) {
        const double s = lane_value(av[n], k);
#pragma unroll
        for (int u = 0; u < RP; ++u) gp[u][n][k & 1] = fma((double)p[u][k], s, gp[u][n][k & 1]);
      }
      if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);   // the next columns of A wait: scalar registers
    }
#pragma unroll
    for (int u = 0; u < RP; ++u)
#pragma unroll
      for (int n = 0; n < NR; ++n)
        if (aa[n][n] > 0.0) {
          double sg = 0.0;
#pragma unroll
          for (int n2 = 0; n2 < NR; ++n2) sg += f[u][n2] * aa[n2][n];
          f[u][n] = row[u] ? fmax(0.0, f[u][n] + (gp[u][n][0] + gp[u][n][1] - sg) / aa[n][n]) : 0.0;
        }
  }
#pragma unroll
  for (int n = 0; n < NR; ++n) {
#pragma unroll
    for (int u = 0; u < RP; ++u)
      if (row[u]) F[(t + 256 * u) * R8 + n] = f[u][n];
    if (wv == 0 && col) A[lane * R8 + n] = av[n];
  }
  __syncthreads();
}

__device__ __forceinline__ void put_word(u64* p, unsigned tag, unsigned half) {
  __hip_atomic_store(p, ((u64)tag << 32) | half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ u64 get_word(u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ROWS: every component is one workgroup's, few segments: half the threads,
// with twice the registers, for the sweeps in registers (hals_rows)
template <bool ROWS>
__global__ __launch_bounds__(ROWS ? 512 : 1024) void k_nmf_split(NmfArgs a, NmfSplit s) {
  constexpr int CT = ROWS ? 512 : 1024, CW = CT / 64;
  constexpr int CV = CT - 64;   // all waves but the last in the HALS product phases (the last: Gram)
  extern __shared__ double dyn[];
  __shared__ double red[CW];
  __shared__ int redi[CW];
  __shared__ double gF[R8 * R8], gA[R8 * R8];
  __shared__ double gpart[64 * R8];   // Gram chunk sums (64 lanes x R8)
  __shared__ int picks[R8];
  __shared__ int bad;
  const int g = blockIdx.x, t = threadIdx.x;
  const int c = s.wg_comp[g];
  const int w0 = s.wg_base[c], nw = s.wg_n[c], r = s.wg_rank[g];
  const int off = a.coff[c], Mc = a.coff[c + 1] - off;
  const int mw = s.mw, lo = r * mw, ml = min(mw, Mc - lo);  // own rows [lo, lo + ml)
  const int K = a.K, Kp = s.Kp, XS = s.XS;
  // LDS: A [K][R8], F [mw][R8], F^T P totals [R8][K], scratch [scr], P rows [mw][Kp] (float)
  double* A = dyn;
  double* F = A + (size_t)K * R8;
  double* FtP = F + (size_t)mw * R8;
  double* scr = FtP + (size_t)R8 * K;
  float* Pl = reinterpret_cast<float*>(scr + s.scr);
  double* R = a.R + (long long)(off + lo) * K;  // own residual rows [ml][K], HBM
  unsigned* abandoned = s.sync + c;
  unsigned* error = s.sync + a.ncomp;
  unsigned ex = 0;  // exchanges done
  bool dead = false;  // this thread gave up waiting (the workgroup leaves at the next check)
  if (t == 0) bad = 0;
  // a component of one workgroup exchanges nothing: what it would put in its
  // slot goes to the LDS words where the totals are wanted (the caller's
  // barriers, or the thread itself, order the accesses)
  const bool alone = ROWS || nw == 1;
  // element j of this workgroup's slot for exchange e
  auto put = [&](unsigned e, size_t j, double v) {
    if (alone) {
      if (j < (size_t)R8 * K) FtP[j] = v;
      else gF[j - (size_t)R8 * K] = v;
      return;
    }
    u64* p = s.xbuf + (((unsigned)(w0 + r) * 2 + (e & 1)) * 2 * (unsigned)XS + (unsigned)j);
    const u64 b = (u64)__double_as_longlong(v);
    put_word(p, e + 1, (unsigned)(b >> 32));
    put_word(p + XS, e + 1, (unsigned)b);
  };
  // sum (or max) of element j over the component's slots of exchange e, in
  // slot order, waiting until each slot's words carry its tag. Up to eight
  // slots are polled together, so that what is late at the first look costs
  // one more round trip for all of them; each late slot polled by itself, with
  // three of four polls at workgroup scope (which the L1 answers from what it
  // read before), made a sweep of 256 x 256 x 3,000 take 16 us instead of 8.
  auto poll = [&](auto count, int wb, unsigned j, unsigned e, bool take_max, double& v) {
    constexpr int C = decltype(count)::value;
    const unsigned tag = e + 1;
    u64 hi[C], lw[C];
    const long long t0 = wall_clock64();
    for (unsigned n = 0;; ++n) {
      // all loads go out before the first use (slots past the last are read
      // as the last one and not used)
#pragma unroll
      for (int q = 0; q < C; ++q) {
        // 32-bit offsets from one base: two addresses per slot held in
        // scalar registers spilled hundreds of them
        const unsigned at = ((unsigned)(w0 + min(wb + q, nw - 1)) * 2 + (e & 1)) * 2 * (unsigned)XS + j;
        hi[q] = get_word(s.xbuf + at);
        lw[q] = get_word(s.xbuf + (at + (unsigned)XS));
      }
#pragma unroll
      for (int q = 0; q < C; ++q) asm volatile("" : "+v"(hi[q]), "+v"(lw[q]));
      unsigned late = 0;
#pragma unroll
      for (int q = 0; q < C; ++q) late |= ((unsigned)(hi[q] >> 32) ^ tag) | ((unsigned)(lw[q] >> 32) ^ tag);
      if (late == 0) break;
      if ((n & 15) == 15 && __hip_atomic_load(abandoned, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
        dead = true;
      } else if (wall_clock64() - t0 > s.limit) {   // no slot comes this late: give the component up
        __hip_atomic_store(abandoned, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        dead = true;
      }
      if (dead) {
        bad = 1;
        return;
      }
    }
#pragma unroll
    for (int q = 0; q < C; ++q)
      if (wb + q < nw) {
        const double x = __longlong_as_double((long long)((hi[q] << 32) | (lw[q] & 0xffffffffull)));
        v = take_max ? fmax(v, x) : v + x;
      }
  };
  auto gather = [&](unsigned j, unsigned e, bool take_max) {
    if (alone) return j < (unsigned)(R8 * K) ? FtP[j] : gF[j - (unsigned)(R8 * K)];
    double v = 0.0;
    for (int wb = 0; wb < nw && !dead;) {
      if (nw - wb > 4) {
        poll(std::integral_constant<int, 8>{}, wb, j, e, take_max, v);
        wb += 8;
      } else {
        poll(std::integral_constant<int, 4>{}, wb, j, e, take_max, v);
        wb += 4;
      }
    }
    return dead ? 0.0 : v;
  };
  __syncthreads();
// leave when any thread of the workgroup gave up waiting (read after a barrier)
#define LEAVE_IF_ABANDONED(ret) \
  __syncthreads();              \
  if (bad) return ret

  // gather own rows: consecutive threads read consecutive pixels of a plane
  for (int e = t; e < ml * K; e += CT) {
    const int i = e / ml, m = e - i * ml;
    Pl[m * Kp + i] = a.p[(long long)i * a.M + a.pix[off + lo + m]];
  }
  __syncthreads();
  for (int e = t; e < ml * K; e += CT) {
    const int m = e / K, i = e - m * K;
    R[e] = (double)Pl[m * Kp + i];
  }
  __syncthreads();

  // ---------------------------------------------------------------- SPA
  double* vec = scr;      // [K] projections
  double* U = scr + K;    // [mw] own entries of the picked direction
  double* nz = A;         // [K] nonzero-column flags (A is free until HALS)
  int N = 0;
  double ref = 0.0;
  while (N < a.max_rank) {
    for (int i = t; i < K; i += CT) {
      {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        int m = 0;
        for (; m + 4 <= ml; m += 4) {
          const double r0 = R[(long long)m * K + i], r1 = R[(long long)(m + 1) * K + i];
          const double r2 = R[(long long)(m + 2) * K + i], r3 = R[(long long)(m + 3) * K + i];
          s0 += r0 * r0;
          s1 += r1 * r1;
          s2 += r2 * r2;
          s3 += r3 * r3;
        }
        for (; m < ml; ++m) {
          const double v = R[(long long)m * K + i];
          s0 += v * v;
        }
        put(ex, i, (s0 + s1) + (s2 + s3));
      }
    }
    double bv = -1.0;
    int bi = INT_MAX;
    for (int i = t; i < K; i += CT) {
      const double sq = gather(i, ex, false);
      if (N == 0) nz[i] = sq > 0.0 ? 1.0 : 0.0;  // the residual is still P (>= 0)
      const double nv = nz[i] > 0.0 ? sqrt(sq) : -1.0;
      if (nv > bv) {
        bv = nv;
        bi = i;
      }
    }
    ++ex;
    LEAVE_IF_ABANDONED();
    double best;
    int j;
    block_argmax<CW>(bv, bi, red, redi, &best, &j);
    if (best <= 0.0) break;
    if (N == 0) ref = best;
    else if (best < a.delta * ref) break;
    if (ROWS && N == kRowsRank) {
      if (t == 0) a.N[c] = kNmfLeft;
      return;
    }
    if (t == 0) picks[N] = j;
    ++N;
    for (int m = t; m < ml; m += CT) U[m] = R[(long long)m * K + j] / best;
    __syncthreads();
    for (int i = t; i < K; i += CT) {
      {
        double s0 = 0.0, s1 = 0.0;
        int m = 0;
        for (; m + 2 <= ml; m += 2) {
          s0 += U[m] * R[(long long)m * K + i];
          s1 += U[m + 1] * R[(long long)(m + 1) * K + i];
        }
        if (m < ml) s0 += U[m] * R[(long long)m * K + i];
        put(ex, i, s0 + s1);
      }
    }
    for (int i = t; i < K; i += CT) {
      vec[i] = gather(i, ex, false);
    }
    ++ex;
    LEAVE_IF_ABANDONED();
    for (int e = t; e < ml * K; e += CT) {
      const int m = e / K, i = e - m * K;
      R[e] -= U[m] * vec[i];
    }
    __syncthreads();
  }
  __syncthreads();

  if (N > 0) {
    // ---------------------------------------------- initial footprints
    for (int n = 0; n < N; ++n) {
      const int col = picks[n];
      double mx = 0.0;
      for (int m = t; m < ml; m += CT) mx = fmax(mx, (double)Pl[m * Kp + col]);
      mx = block_max<CW>(mx, red);
      if (t == 0) put(ex, n, mx);
    }
    if (alone) __syncthreads();
    for (int m = t; m < ml; m += CT)
      for (int n = 0; n < R8; ++n) {
        double v = 0.0;
        if (n < N) {
          v = (double)Pl[m * Kp + picks[n]] / gather(n, ex, true);
        }
        F[m * R8 + n] = v;
      }
    ++ex;
    for (int e = t; e < K * R8; e += CT) A[e] = 0.0;
    LEAVE_IF_ABANDONED();

    if constexpr (ROWS) {
      const int kc = (K + N + 15) / 16;
      auto in_rows = [&](auto rank, auto per) {
        constexpr int NR = decltype(rank)::value, RP = decltype(per)::value;
        if (kc == 1) hals_rows<RP, NR, 1>(Pl, Kp, F, A, scr, ml, K, a.sweeps);
        else if (kc == 2) hals_rows<RP, NR, 2>(Pl, Kp, F, A, scr, ml, K, a.sweeps);
        else hals_rows<RP, NR, 3>(Pl, Kp, F, A, scr, ml, K, a.sweeps);
      };
      auto by_rank = [&](auto per) {
        if (N == 1) in_rows(std::integral_constant<int, 1>{}, per);
        else if (N == 2) in_rows(std::integral_constant<int, 2>{}, per);
        else in_rows(std::integral_constant<int, 3>{}, per);
      };
      if (ml <= 256) by_rank(std::integral_constant<int, 1>{});
      else by_rank(std::integral_constant<int, 2>{});
    } else {
      // HALS, compiled per rank so that the sequential row/column updates run
      // without predication
      auto hals = [&](auto rank) -> bool {
        constexpr int NR = decltype(rank)::value;
        constexpr int NP = NR * (NR + 1) / 2;
        for (int sweep = -1; sweep < a.sweeps; ++sweep) {
          // ---- partial F^T P and F^T F over own rows (FP64, fixed order),
          // written to this workgroup's slot. Waves 0..14: thread (row chunk
          // q, segment i) sums its rows for all NR columns of F; after the
          // barrier the chunks are added in order and written to the slot,
          // and the gather of the totals follows without another barrier.
          // Wave 15: F^T F, whole within the wave (gram_wave), straight to the
          // slot.
          {
            // chunks of about 16 rows, at least 8 and at most 24 of them
            const int QC = max(1, min(min(CV / K, max(8, min(24, ml / 16))), s.scr / (K * NR)));
            const int rows = (ml + QC - 1) / QC;
            if (t < CV) {
              for (int e = t; e < QC * K; e += CV) {
                const int q = e / K, i = e - q * K;
                const int m1 = min(ml, (q + 1) * rows);
                double s0[NR], s1[NR];
#pragma unroll
                for (int n = 0; n < NR; ++n) s0[n] = s1[n] = 0.0;
                int m = q * rows;
                if constexpr (NR <= 3) {   // four rows' reads in flight
                  for (; m + 3 < m1; m += 4) {
                    double p[4], f[4][NR];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                      p[u] = (double)Pl[(m + u) * Kp + i];
#pragma unroll
                      for (int n = 0; n < NR; ++n) f[u][n] = F[(m + u) * R8 + n];
                    }
#pragma unroll
                    for (int n = 0; n < NR; ++n) {
                      s0[n] = fma(f[0][n], p[0], s0[n]);
                      s1[n] = fma(f[1][n], p[1], s1[n]);
                      s0[n] = fma(f[2][n], p[2], s0[n]);
                      s1[n] = fma(f[3][n], p[3], s1[n]);
                    }
                  }
                }
                for (; m + 1 < m1; m += 2) {
                  const double p0 = (double)Pl[m * Kp + i], p1 = (double)Pl[(m + 1) * Kp + i];
#pragma unroll
                  for (int n = 0; n < NR; ++n) {
                    s0[n] = fma(F[m * R8 + n], p0, s0[n]);
                    s1[n] = fma(F[(m + 1) * R8 + n], p1, s1[n]);
                  }
                }
                if (m < m1) {
                  const double p0 = (double)Pl[m * Kp + i];
#pragma unroll
                  for (int n = 0; n < NR; ++n) s0[n] = fma(F[m * R8 + n], p0, s0[n]);
                }
#pragma unroll
                for (int n = 0; n < NR; ++n) {
                  if (QC == 1) put(ex, (size_t)n * K + i, s0[n] + s1[n]);
                  else scr[(size_t)e * NR + n] = s0[n] + s1[n];
                }
              }
            } else {   // F^T F of the own rows, upper triangle
              const double v = gram_wave<NR>(F, ml, t - CV, gpart);
              if (t - CV < NP) {
                int n1, n2;
                pair_of<NR>(t - CV, n1, n2);
                put(ex, (size_t)R8 * K + n1 * R8 + n2, v);
              }
            }
            __syncthreads();
            if (QC > 1)
              for (int o = t; o < NR * K; o += CT) {
                const int n = o / K, i = o - n * K;
                put(ex, o, chunk_sum(scr + (size_t)i * NR + n, (size_t)K * NR, QC));
              }
          }
          // ---- totals over the component's workgroups (slot order) into LDS:
          // the NR K entries of F^T P, then the upper triangle of F^T F (mirrored)
          for (int e = t; e < NR * K + NP; e += CT) {
            if (e < NR * K) {
              if (!alone) FtP[e] = gather(e, ex, false);
            } else {
              int n1, n2;
              pair_of<NR>(e - NR * K, n1, n2);
              const double v = gather((unsigned)(R8 * K + n1 * R8 + n2), ex, false);
              gF[n1 * R8 + n2] = v;
              gF[n2 * R8 + n1] = v;
            }
          }
          ++ex;
          LEAVE_IF_ABANDONED(false);
          // ---- the A update (rows of A in order), every workgroup alike
          for (int i = t; i < K; i += CT) {
            double av[NR];
#pragma unroll
            for (int n = 0; n < NR; ++n) av[n] = A[i * R8 + n];
#pragma unroll
            for (int n = 0; n < NR; ++n) {
              // from rank 6 on, hoisting all Gram reads would spill: keep them per row
              if constexpr (NR > 5) asm volatile("" ::: "memory");
              const double d = gF[n * R8 + n];
              if (d > 0.0) {
                double sg = 0.0;
#pragma unroll
                for (int n2 = 0; n2 < NR; ++n2) sg += gF[n * R8 + n2] * av[n2];
                av[n] = fmax(0.0, av[n] + (FtP[n * K + i] - sg) / d);
              }
            }
#pragma unroll
            for (int n = 0; n < NR; ++n) A[i * R8 + n] = av[n];
          }
          __syncthreads();
          if (sweep < 0) continue;
          // ---- P A^T of own rows and A A^T (FP64, fixed order). Waves
          // 0..14: thread (segment chunk q, own row m) sums its segments for
          // all NR rows of A. Wave 15: A A^T whole within the wave, chunked by
          // K and NR only, so identical in every workgroup.
          // at most 16 chunks: their in-order sum is a chain of dependent adds
          const int QK = max(1, min(min(CV / ml, 16), s.scr / (ml * NR)));
          {
            const int seg = (K + QK - 1) / QK;
            if (t < CV) {
              for (int e = t; e < QK * ml; e += CV) {
                const int q = e / ml, m = e - q * ml;
                const int i1 = min(K, (q + 1) * seg);
                double s0[NR], s1[NR];
#pragma unroll
                for (int n = 0; n < NR; ++n) s0[n] = s1[n] = 0.0;
                int i = q * seg;
                for (; i + 1 < i1; i += 2) {
                  const double p0 = (double)Pl[m * Kp + i], p1 = (double)Pl[m * Kp + i + 1];
#pragma unroll
                  for (int n = 0; n < NR; ++n) {
                    s0[n] = fma(p0, A[i * R8 + n], s0[n]);
                    s1[n] = fma(p1, A[(i + 1) * R8 + n], s1[n]);
                  }
                }
                if (i < i1) {
                  const double p0 = (double)Pl[m * Kp + i];
#pragma unroll
                  for (int n = 0; n < NR; ++n) s0[n] = fma(p0, A[i * R8 + n], s0[n]);
                }
#pragma unroll
                for (int n = 0; n < NR; ++n) scr[(size_t)e * NR + n] = s0[n] + s1[n];
              }
            } else {   // A A^T, upper triangle mirrored (every workgroup alike)
              const double v = gram_wave<NR>(A, K, t - CV, gpart);
              if (t - CV < NP) {
                int n1, n2;
                pair_of<NR>(t - CV, n1, n2);
                gA[n1 * R8 + n2] = v;
                gA[n2 * R8 + n1] = v;
              }
            }
            __syncthreads();
          }
          // ---- the own F rows (columns of F in order), each thread adding
          // its row's P A^T chunks in order first
          for (int m = t; m < ml; m += CT) {
            double gp[NR], f[NR];
#pragma unroll
            for (int n = 0; n < NR; ++n) {
              gp[n] = chunk_sum(scr + (size_t)m * NR + n, (size_t)ml * NR, QK);   // P A^T: chunks in order
              f[n] = F[m * R8 + n];
            }
#pragma unroll
            for (int n = 0; n < NR; ++n) {
              if constexpr (NR > 5) asm volatile("" ::: "memory");
              const double d = gA[n * R8 + n];
              if (d > 0.0) {
                double sg = 0.0;
#pragma unroll
                for (int n2 = 0; n2 < NR; ++n2) sg += f[n2] * gA[n2 * R8 + n];
                f[n] = fmax(0.0, f[n] + (gp[n] - sg) / d);
              }
            }
#pragma unroll
            for (int n = 0; n < NR; ++n) F[m * R8 + n] = f[n];
          }
          __syncthreads();
        }
        return true;
      };
      bool ok = true;
      switch (N) {
        case 1: ok = hals(std::integral_constant<int, 1>{}); break;
        case 2: ok = hals(std::integral_constant<int, 2>{}); break;
        case 3: ok = hals(std::integral_constant<int, 3>{}); break;
        case 4: ok = hals(std::integral_constant<int, 4>{}); break;
        case 5: ok = hals(std::integral_constant<int, 5>{}); break;
        case 6: ok = hals(std::integral_constant<int, 6>{}); break;
        case 7: ok = hals(std::integral_constant<int, 7>{}); break;
        default: ok = hals(std::integral_constant<int, 8>{}); break;
      }
      if (!ok) return;
    }

    // ------------------------------------------ scale to peak 1, export
    for (int n = 0; n < N; ++n) {
      double mx = 0.0;
      for (int m = t; m < ml; m += CT) mx = fmax(mx, F[m * R8 + n]);
      mx = block_max<CW>(mx, red);
      if (t == 0) put(ex, n, mx);
    }
    double* peak = scr;
    if (alone) __syncthreads();
    if (t < N) peak[t] = gather(t, ex, true);
    ++ex;
    LEAVE_IF_ABANDONED();
    double* Fg = a.F + (long long)(off + lo) * R8;
    double* Ag = a.A + (long long)c * R8 * a.Kmax;
    for (int n = 0; n < N; ++n) {
      const double sc = peak[n] > 0.0 ? peak[n] : 1.0;
      for (int m = t; m < ml; m += CT) Fg[(long long)m * R8 + n] = F[m * R8 + n] / sc;
      if (r == 0)
        for (int i = t; i < K; i += CT) Ag[(long long)n * a.Kmax + i] = A[i * R8 + n] * sc;
    }
  }
#undef LEAVE_IF_ABANDONED
  if (r == 0 && t == 0) a.N[c] = N;
}

__global__ void k_fill_u32(unsigned* p, int n, unsigned v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Dynamic LDS of one workgroup: A [K][R8], F [mw][R8], F^T P totals [R8][K],
// scratch (the chunk partials of the HALS products, the SPA vectors, the final
// column maxima or the waves' sums of the sweeps in registers), P rows
// [mw][Kp]. The HALS products need a double per row and rank at least: slices
// of up to kSliceMax rows have that at every rank. (The sweeps in registers
// need rows_scratch, whatever their rows.)
constexpr int kSliceMax = 192, kScratch = kSliceMax * R8;
static_assert(rows_scratch(kRowsK) <= kScratch, "the waves' sums fit the scratch");
size_t split_lds(int K, int mw, int* scr_out) {
  const int Kp = K | 1;
  const size_t scr = std::max<size_t>({(size_t)kScratch, (size_t)K + mw});
  if (scr_out) *scr_out = (int)scr;
  return 8 * ((size_t)K * R8 + (size_t)mw * R8 + (size_t)R8 * K + scr) + 4 * (size_t)mw * Kp;
}

}  // namespace

bool plan_nmf_split(NmfSplit& s, const NmfArgs& a, const std::vector<int>& coff, const int* ranks, size_t xbuf_bytes,
                    NmfSplitTables& tab) {
  int dev = 0, coop = 0, ncu = 0, max_lds = 0, clock_khz = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop)
    return false;
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
  if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
    return false;
  if (hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || clock_khz <= 0)
    return false;
  const size_t budget = max_lds > 16384 ? (size_t)max_lds - 12288 : 0;  // static LDS ~1.3 KB, with room to spare
  const int K = a.K;
  const int ncomp = a.ncomp;
  if (K < 1 || ncomp < 1) return false;
  const int XS = ((R8 * K + R8 * R8) + 31) / 32 * 32;
  // exchange slots: two per workgroup of the largest launch, in xbuf, each
  // of XS high and XS low words
  const size_t slot_bytes = (size_t)2 * 2 * XS * 8;
  // pixels of component k that this plan takes (none of one that is done)
  auto pixels = [&](int k) { return ranks && ranks[k] != kNmfLeft ? 0 : coff[k + 1] - coff[k]; };
  // Slice widths in order of preference: 96 rows balance the per-sweep exchange
  // against the per-workgroup work where there are many segments, 160 where
  // there are few and a row is little work (at 60 segments 1.64 ms against
  // 1.86 for 96 rows and 1.81 for 208; at 90 2.34 against 2.39; at 120 1.79
  // against 1.54). Components are packed, in order, into launches of at most
  // one workgroup per compute unit; each launch costs about the same (its
  // sweeps are latency bound), so the width with the fewest launches wins.
  const bool few = K <= 96;
  const int widths[] = {few ? 160 : 96, 128, few ? 96 : 160, kSliceMax, 64, 32};
  int mw = 0, best_groups = 0;
  for (const int w : widths) {
    if (split_lds(K, w, nullptr) > budget) continue;
    int groups = 1, in_group = 0, widest = 0;
    bool fits = true;
    for (int k = 0; k < ncomp && fits; ++k) {
      const int nwk = (pixels(k) + w - 1) / w;
      if (nwk > ncu) fits = false;
      else if (in_group + nwk > ncu) {
        ++groups;
        in_group = nwk;
      } else {
        in_group += nwk;
      }
      widest = std::max(widest, in_group);
    }
    fits = fits && (size_t)widest * slot_bytes <= xbuf_bytes;
    if (fits && (mw == 0 || groups < best_groups)) {
      mw = w;
      best_groups = groups;
    }
  }
  if (mw == 0) return false;
  // Short recordings whose components all fit one workgroup each take the
  // sweeps in registers (0.25 ms against 0.86 at 8 segments, 0.32 against 0.90
  // at 20, in registers first; 48 columns and the Gram entries are what the
  // registers hold, and 512 rows of P_c and F what the LDS does). Components
  // that they leave have a plan of the other kind, since one was found above.
  int most = 0;
  for (int k = 0; k < ncomp; ++k) most = std::max(most, pixels(k));
  const int one = (most + 63) / 64 * 64;
  s.rows = !ranks && K <= kRowsK && most <= kRowsMax && split_lds(K, one, nullptr) <= budget;
  if (s.rows) mw = one;
  int scr = 0;
  size_t lds = split_lds(K, mw, &scr);
  if (!s.rows) {
    if (scr < mw * R8) return false;   // a double per row and rank for the HALS products
    // spare LDS (up to 3 R8 K more doubles) widens the scratch of the HALS
    // products' chunk partials, so more chunks run at once at higher ranks
    const size_t more = std::min<size_t>((budget - lds) / 8, (size_t)3 * R8 * K);
    scr += (int)more;
    lds += 8 * more;
  }
  int occ = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, s.rows ? k_nmf_split<true> : k_nmf_split<false>,
                                                   s.rows ? 512 : 1024, lds) != hipSuccess || occ < 1)
    return false;
  s.mw = mw;
  s.Kp = K | 1;
  s.scr = scr;
  s.XS = XS;
  s.lds_bytes = lds;
  s.limit = (long long)clock_khz * 1000LL * 2;  // two seconds of wall clock
  tab.comp.clear();
  tab.rank.clear();
  tab.base.assign((size_t)ncomp, 0);
  tab.n.assign((size_t)ncomp, 0);
  tab.groups.clear();
  // components in order into launches; base[k] numbers a component's slots
  // within its launch
  std::vector<std::vector<int>> members(1);
  int start = 0, in_group = 0;
  for (int k = 0; k < ncomp; ++k) {
    const int nwk = (pixels(k) + mw - 1) / mw;
    if (in_group + nwk > ncu) {
      tab.groups.push_back({start, in_group});
      members.emplace_back();
      start += in_group;
      in_group = 0;
    }
    tab.base[k] = in_group;
    tab.n[k] = nwk;
    members.back().push_back(k);
    in_group += nwk;
  }
  tab.groups.push_back({start, in_group});
  // Workgroup g of a launch runs on XCD g mod 8 (the dispatcher deals
  // workgroups to the XCDs in turn). Each component gets workgroups of one
  // XCD where one has room (largest components first, into the XCD with the
  // most room), so its exchanges stay in that XCD's L2; the rest take what
  // is left.
  constexpr int NX = 8;
  tab.comp.assign((size_t)start + in_group, 0);
  tab.rank.assign((size_t)start + in_group, 0);
  for (size_t gi = 0; gi < tab.groups.size(); ++gi) {
    const int first = tab.groups[gi].first, G = tab.groups[gi].second;
    std::vector<std::vector<int>> free_g(NX);
    for (int g = G - 1; g >= 0; --g) free_g[g % NX].push_back(g);   // popped in increasing order
    std::vector<int> order = members[gi];
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return tab.n[x] > tab.n[y]; });
    std::vector<int> spill;
    for (const int k : order) {
      int best = -1;
      for (int x = 0; x < NX; ++x)
        if ((int)free_g[x].size() >= tab.n[k] && (best < 0 || free_g[x].size() > free_g[best].size())) best = x;
      if (best < 0) {
        spill.push_back(k);
        continue;
      }
      for (int j = 0; j < tab.n[k]; ++j) {
        const int g = free_g[best].back();
        free_g[best].pop_back();
        tab.comp[first + g] = k;
        tab.rank[first + g] = j;
      }
    }
    for (const int k : spill)
      for (int j = 0, x = 0; j < tab.n[k]; ++j) {
        while (free_g[x].empty()) ++x;
        const int g = free_g[x].back();
        free_g[x].pop_back();
        tab.comp[first + g] = k;
        tab.rank[first + g] = j;
      }
  }
  s.G = (int)tab.comp.size();
  return true;
}

hipError_t launch_nmf_split(const NmfArgs& a, const NmfSplit& s, bool first, hipStream_t st) {
  hipError_t e = hipSuccess;
  if (first) {   // the abandon flags of every component and the error flag, once per plan
    const int nsync = a.ncomp + 1;
    hipLaunchKernelGGL(k_fill_u32, dim3((nsync + 255) / 256), dim3(256), 0, st, s.sync, nsync, 0u);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const void* kernel = reinterpret_cast<const void*>(s.rows ? k_nmf_split<true> : k_nmf_split<false>);
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds_bytes);
  if (e != hipSuccess) return e;
  if (s.rows) {   // nothing is exchanged
    hipLaunchKernelGGL(k_nmf_split<true>, dim3(s.G), dim3(512), (unsigned)s.lds_bytes, st, a, s);
    return hipGetLastError();
  }
  {   // the slots of this launch carry no tag (tags start at 1)
    const long long words = (long long)s.G * 2 * 2 * s.XS * 2;   // 32-bit words
    if (words > INT_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<unsigned*>(s.xbuf), (int)words, 0u);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  NmfArgs aa = a;
  NmfSplit ss = s;
  void* args[] = {&aa, &ss};
  return hipLaunchCooperativeKernel(kernel, dim3(s.G), dim3(1024), args, (unsigned)s.lds_bytes, st);
}

}  // namespace seg
