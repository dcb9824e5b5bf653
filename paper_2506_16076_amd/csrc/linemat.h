// Line derivatives as matrix products on the fp16 matrix cores, at FP32
// accuracy (lines of up to 512 samples, 640 with their continuation).
//
// The FC derivative of a line is K Delta ext: Delta ext the L cyclic first
// differences of the extension (engine.h), K the N x L section of the
// circulant with first column
//     kappa[m] = (1/L) sum_k w_k cos(2 pi k (m - 1/2) / L) / sin(pi k / L),
// k = 1 .. (L-1)/2, w_k = 2 pi k / (L h): the multipliers i w_k /
// (exp(2 pi i k/L) - 1) of the transform, summed in closed form.  Reversing
// the line maps Delta ext[n] to -Delta ext[N-2-n] and the derivative to its
// negative, so K[N-1-i][N-2-n] = K[i][n] and one product of the full size
// becomes two of half the rows and half the columns: with the pairs (n, n' =
// N-2-n mod L) of differences, xe = x_n + x_n', xo = x_n - x_n',
//     out_i = E_i + O_i,  out_{N-1-i} = E_i - O_i,
//     E = Me xe, O = Mo xo, Me = (K_n + K_n') / 2, Mo = (K_n - K_n') / 2.
// Pair slots: the differences of the samples at 0 .. Ni - 1, Ni = N/2, the C + 1
// differences that involve the tail (FP64 rows applied to the end samples) at
// Ni .. Ni + (C+2)/2 - 1; zero up to the next multiple of 32.
//
// Operands: v = hi + lo, hi = fp16(v), lo = fp16(v - hi), 22-23 significant
// bits; hi hi + lo hi + hi lo of every pair are summed in FP32 accumulators of
// the 16x16x32 products (lo lo is below 2^-22 of a term).  A column is scaled
// by a power of two from its largest operand xe, xo (the tail's among them)
// into the top of the fp16 range, the table once per plan, so lo needs no scale
// of its own: it rounds to zero only below 2^-39 of the largest operand.  (A
// scale from the largest sample loses as many of these bits as the sample is
// larger than its differences.)
// Error against 64 bits, relative to the derivative's L2 norm (lines of 48 ..
// 512 samples, d = 2 and 5), products and FP32 transform:
//   1.4 (1 + a sin), a = 1 .. 1e-3:  1.2e-7 .. 2.0e-7   1.5e-7 .. 3.0e-7
//   a = 1e-5, 1e-6, d = 2:           0.9e-7 .. 1.5e-7   1.5e-7 .. 4.5e-7
//   a = 1e-5, 1e-6, d = 5:           3e-7 .. 4e-6       1.5e-6 .. 3e-5
//   noise, d = 2:                    1.2e-7 .. 2.1e-7   1.4e-7 .. 1.6e-7
//   noise, d = 5:                    2e-6 .. 7e-6       2e-5 .. 4e-5
// (noise with d = 2 on lines from 256 samples on is the one kind where the
// transform is nearer: the products' running sums are rounded once a block of
// 32 pairs and partial product.)
//
// What bounds it: per value L multiply-adds times three partial products, 0.2
// ms per 15.8 M point stage at the dense fp16 rate, and the table, streamed
// from L2 once per tile (about L/16 bytes a value).  Of the fused q2 pass's
// 768 us (15.8 M points, one workgroup size for all lines) its loads and
// stores alone took 414, splitting and tail 54, the products without the
// table's loads 130, those 170: against the transform's 724 the final pass
// takes 703.  Where sets are small the transform's many short phases are
// latency: the right-hand side of 24 patches with C = 27 on every line 631 ->
// 342 us, a step of one 64 x 64 patch 779 -> 265 us.
#pragma once
#include "kernels.h"

namespace fcsd {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float mfloat4;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 mhalf8;

// Two sizes of lines, each with its own kernels.  Workgroups are as small as
// their LDS lets a compute unit hold 16 waves: several of them overlap one
// tile's memory phases with another's arithmetic, and a thread has enough
// elements to pay for a phase's fixed work.  A thread folds at most `items`
// octets of pairs (kept in registers across a barrier), a wave multiplies at
// most `rows` row blocks of the table, reading it `ahead` half K steps ahead;
// `waves` per SIMD bound the registers.
struct MatSmall {  // up to 256 samples
  static constexpr int threads = 256, items = 3, rows = 2, ahead = 2, waves = 4, load = 6, epiH = 4, epiC = 4;
};
struct MatLarge {  // up to 512 samples
  static constexpr int threads = 512, items = 3, rows = 2, ahead = 2, waves = 4, load = 6, epiH = 4, epiC = 4;
};
#define FCSD_MAT_BOUNDS(CLS) __launch_bounds__(CLS::threads, CLS::waves)

// LDS of a tile, in 32-bit words: two halves (first members of the pairs,
// then the second), each KR = 8 KS rows of four slots x columns: slot n,
// column c at (n/4) ldw + 4 (c ^ x) + n%4, x = 4 in odd rows (tiles of 32
// columns on: the eight samples x four lines that half a wave stores lie in
// distinct banks).  Samples f_i take slot i of the first half, i < Nh =
// (N+1)/2, else slot N-1-i of the second; so do the results.  The split
// operands of eight pairs take the eight places of their slots: the row pair's
// first row the hi halves, the second the lo halves.  Then the column maxima
// and one word per column for the first tail difference of an odd line, whose
// place its middle sample holds.  The FP64 rows of the tail differences come
// last.
__host__ __device__ __forceinline__ size_t mat_lds_bytes(int ks, int ncp, int C, int d) {
  return 4 * ((size_t)16 * ks * 4 * ncp + 2 * (size_t)ncp) + 16 * (size_t)(C ? C + 1 : 0) * d;
}

struct MatCtx {
  unsigned* z;
  unsigned* cmax;  // [ncp]: bits of each column's largest operand
  float* side;     // [ncp]
  double* dq;      // [C + 1][2 d]
  int ncp, lgc;    // columns (16 or 32) and their log2: F fields x (ncp / F) lines, column f ncp/F + line
  int lgn;         // log2 of the lines
  int ldw, hs;     // row stride, offset of the second half
  int KO, N, Nh, Ni, Pt;

  __device__ __forceinline__ int odd_row(int row) const { return ncp > 16 ? 4 * (row & 1) : 0; }
  // word of slot n of line `line`, field 0 (field f: 4 f ncp/F further)
  __device__ __forceinline__ int word(int n, int line) const {
    return (n >> 2) * ldw + (n & 3) + 4 * (line ^ odd_row(n >> 2));
  }
};

// The thread's index, opaque to the compiler: what a round computes from it is
// not hoisted out of the loop over the rounds (where its addresses would be
// held, and spilled, across the matrix products).
__device__ __forceinline__ int mat_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ float* lds_f(unsigned* z) { return reinterpret_cast<float*>(z); }

template <int F = 4>
__device__ __forceinline__ MatCtx mat_setup(unsigned* lds, const PassArgs& a, const PlanDev& P, int ncp) {
  MatCtx X;
  X.z = lds;
  X.ncp = ncp;
  X.lgc = 31 - __builtin_clz(ncp);
  X.lgn = X.lgc - (F == 4 ? 2 : 1);
  X.ldw = 4 * ncp;
  X.KO = 4 * P.mks;
  X.hs = 2 * X.KO * X.ldw;
  X.cmax = lds + 2 * X.hs;
  X.side = lds_f(X.cmax + ncp);
  X.N = P.N;
  X.Nh = (P.N + 1) >> 1;
  X.Ni = P.N >> 1;
  X.Pt = (P.C + 2) >> 1;
  X.dq = reinterpret_cast<double*>(X.side + ncp);
  if (!P.periodic)
    for (int i = threadIdx.x; i < (P.C + 1) * 2 * a.d; i += blockDim.x) X.dq[i] = a.dq[P.dq + i];
  return X;
}

// A thread's elements of a tile: blocks of 32 stored ones (PB positions x LB
// lines: a block of the blocked storage; 32 samples of one line, or 8 lines x
// 4, of the row-major one), taken so that the thread keeps its line and its
// row parity: byte offset from the tile's first stored element and both words
// (as a sample of the first half, and of the second) advance by constants.
struct MatThread {
  int pos, stop, line;  // first position, end (0: the thread's line is not in the tile)
  int wa, wb, dpos, dw;
  unsigned g, dg;
};

template <int DIR>
__device__ __forceinline__ MatThread mat_thread(const MatCtx& X, const PlanDev& P, int nl) {
  MatThread M;
  const int t = threadIdx.x, w = t & 31, slot = t >> 5;
  int ln, pi, lgl, lgp;  // line and position in the block, log2 of LB and PB
  unsigned g, gpb, glg;  // byte offset, steps from block to block along the line, from line group to line group
  if (P.nb1) {
    g = 4u * w;
    if (DIR == 1) {
      lgl = 2, lgp = 3, pi = w & 7, ln = w >> 3;
      gpb = 128u, glg = 128u * P.nb1;
    } else {
      lgl = 3, lgp = 2, pi = w >> 3, ln = w & 7;
      gpb = 128u * P.nb1, glg = 128u;
    }
  } else if (DIR == 1) {
    lgl = 0, lgp = 5, pi = w, ln = 0;
    g = 4u * w, gpb = 128u, glg = 4u * P.n1;
  } else {
    lgl = 3, lgp = 2, pi = w >> 3, ln = w & 7;
    g = 4u * (unsigned)(pi * P.n1 + ln), gpb = 16u * P.n1, glg = 32u;
  }
  // line groups: a power of two, no more than the workgroup's 32-thread slots
  const int lgG = max(X.lgn - lgl, 0);
  const int lg = slot & ((1 << lgG) - 1), PS = (int)(blockDim.x >> 5) >> lgG;
  M.line = (lg << lgl) + ln;
  M.stop = M.line < nl ? X.N : 0;
  M.pos = ((slot >> lgG) << lgp) + pi;
  M.dpos = PS << lgp;
  M.dw = (M.dpos >> 2) * X.ldw;
  M.g = g + (unsigned)lg * glg + (unsigned)(slot >> lgG) * gpb;
  M.dg = (unsigned)PS * gpb;
  M.wa = X.word(M.pos, M.line);
  M.wb = X.word(X.N - 1 - M.pos, M.line) + X.hs;
  return M;
}

// Visit the thread's elements in batches of U: pre(g) issues the loads of every
// element of the batch (elements past the tile read its first one), post(g, w,
// value) consumes the valid ones; w: the word of field 0 in LDS.
template <int U, class Pre, class Post>
__device__ __forceinline__ void mat_walk(const MatCtx& X, const MatThread& M, Pre&& pre, Post&& post) {
  using T = decltype(pre(0u));
  int pos = M.pos, wa = M.wa, wb = M.wb;
  unsigned g = M.g;
  asm volatile("" : "+v"(pos));  // addresses of a batch are formed where they are used, not kept over the rounds
  for (; pos < M.stop; pos += U * M.dpos) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = pre(pos + u * M.dpos < X.N ? g + u * M.dg : 0u);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (pos + u * M.dpos < X.N)
        post(g + u * M.dg, pos + u * M.dpos < X.Nh ? wa + u * M.dw : wb - u * M.dw, v[u]);
    g += U * M.dg;
    wa += U * M.dw;
    wb -= U * M.dw;
  }
}

// Load four fields of the tile (A0 .. A3 at its first stored element) into the
// sample places.
template <class CLS>
__device__ __forceinline__ void mat_load4(const MatCtx& X, const MatThread& M, const float* A0, const float* A1,
                                          const float* A2, const float* A3) {
  float* z = lds_f(X.z);
  const int ncp = X.ncp;
  mat_walk<CLS::load>(
      X, M, [&](unsigned g) { return make_float4(at(A0, g), at(A1, g), at(A2, g), at(A3, g)); },
      [&](unsigned, int w, float4 v) {
        float* p = z + w;
        p[0] = v.x;
        p[ncp] = v.y;
        p[2 * ncp] = v.z;
        p[3 * ncp] = v.w;
      });
}

// Exponent s of a column's scale 2^s, which takes its largest operand below
// 2^15.  A column with an infinity or NaN stays unscaled (its results are not
// finite either way).
__device__ __forceinline__ int mat_scale(unsigned bits) {
  const int E = (int)(bits >> 23);
  return E == 255 ? 0 : min(141 - E, 126);
}

// The fp16 halves of two values scaled by sc (a power of two): hi, and what it
// leaves, lo.  hi is kept packed and opaque: lo is then one mixed-precision
// FMA a value.
__device__ __forceinline__ void mat_split2(float a, float b, float sc, unsigned& hi, unsigned& lo) {
  typedef __attribute__((__vector_size__(2 * sizeof(_Float16)))) _Float16 half2v;
  half2v h = {(_Float16)(a * sc), (_Float16)(b * sc)};
  __builtin_memcpy(&hi, &h, 4);
  asm("" : "+v"(hi));
  __builtin_memcpy(&h, &hi, 4);
  const half2v l = {(_Float16)fmaf(a, sc, -(float)h[0]), (_Float16)fmaf(b, sc, -(float)h[1])};
  __builtin_memcpy(&lo, &l, 4);
}

__device__ __forceinline__ mhalf8 mat_half8(const uint4& v) {
  mhalf8 h;
  __builtin_memcpy(&h, &v, 16);
  return h;
}

// Products of TR row blocks (16 position pairs each, from rb0) with TC column
// blocks (16 columns): acc[tr][e/o][tc].  The table comes from
// L2 (or beyond, for the first tile of a patch on its die), a latency of one or
// two thousand cycles under the passes' own traffic: its words are read D half
// K steps (the even or the odd part) ahead.  Row blocks past RB repeat
// the last one (not stored).
template <int TR, int TC, int D>
__device__ __forceinline__ void mat_gemm(const uint4* __restrict__ tab, int KS, int rb0, int RB, const MatCtx& X,
                                         mfloat4 (&acc)[TR][2][TC]) {
  const int lane = mat_tid() & 63;
  const unsigned lo16 = 16u * lane;
  const uint4* ap[TR];  // uniform
  uint4 a[D][TR][2];
  const int last = 2 * KS - 1;  // half steps 0 .. last
#pragma unroll
  for (int r = 0; r < TR; ++r) ap[r] = tab + (size_t)min(rb0 + r, RB - 1) * KS * 256;
#pragma unroll
  for (int j = 0; j < D; ++j)
#pragma unroll
    for (int r = 0; r < TR; ++r)
#pragma unroll
      for (int p = 0; p < 2; ++p) a[j][r][p] = at(ap[r] + 128 * min(j, last) + 64 * p, lo16);
#pragma unroll
  for (int r = 0; r < TR; ++r)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < TC; ++c) acc[r][h][c] = mfloat4{0.f, 0.f, 0.f, 0.f};
  const int col = lane & 15, ldw = X.ldw;
  const unsigned* bh = X.z + 2 * (lane >> 4) * ldw + 4 * col;
  const unsigned* bl = X.z + (2 * (lane >> 4) + 1) * ldw + 4 * (col ^ X.odd_row(1));
  for (int s0 = 0; s0 <= last; s0 += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int h = j & 1;
      mhalf8 b[2][TC];
#pragma unroll
      for (int c = 0; c < TC; ++c) {
        b[0][c] = mat_half8(*reinterpret_cast<const uint4*>(bh + (h ? X.hs : 0) + 64 * c));
        b[1][c] = mat_half8(*reinterpret_cast<const uint4*>(bl + (h ? X.hs : 0) + 64 * c));
      }
#pragma unroll
      for (int m = 0; m < 3; ++m)  // hi hi, lo hi, hi lo
#pragma unroll
        for (int r = 0; r < TR; ++r)
#pragma unroll
          for (int c = 0; c < TC; ++c)
            acc[r][h][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(mat_half8(a[j][r][m == 1]), b[m == 2][c],
                                                                  acc[r][h][c], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < TR; ++r)
#pragma unroll
        for (int p = 0; p < 2; ++p) a[j][r][p] = at(ap[r] + 128 * min(s0 + j + D, last) + 64 * p, lo16);
      if (h) {
        bh += 8 * ldw;
        bl += 8 * ldw;
      }
    }
  }
}

template <int TR, int TC, int D>
__device__ __forceinline__ void mat_product(const MatCtx& X, const PlanDev& P, const uint4* __restrict__ mt) {
  const int tid = mat_tid(), lane = tid & 63;
  // TR row blocks per wave, all columns
  const int RB = P.mrb, rb0 = __builtin_amdgcn_readfirstlane(tid >> 6) * TR;
  const bool on = rb0 < RB;
  mfloat4 acc[TR][2][TC];
  if (on) mat_gemm<TR, TC, D>(mt + P.mt, P.mks, rb0, RB, X, acc);
  __syncthreads();  // every operand has been read: the results take their places
  if (on) {
    const unsigned* cm = X.cmax;
    float* z = lds_f(X.z);
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      const int col = 16 * c + (lane & 15);
      const int e = -(mat_scale(cm[col]) + P.mes);
      float* oc = z + (4 * rb0 + (lane >> 4)) * X.ldw + 4 * (col ^ X.odd_row(lane >> 4));
#pragma unroll
      for (int r = 0; r < TR; ++r) {
        if (rb0 + r >= RB) continue;
        float* o = oc + 4 * r * X.ldw;
        const mfloat4 E = acc[r][0][c], O = acc[r][1][c];
        *reinterpret_cast<float4*>(o) = make_float4(ldexpf(E[0] + O[0], e), ldexpf(E[1] + O[1], e),
                                                    ldexpf(E[2] + O[2], e), ldexpf(E[3] + O[3], e));
        *reinterpret_cast<float4*>(o + X.hs) = make_float4(ldexpf(E[0] - O[0], e), ldexpf(E[1] - O[1], e),
                                                           ldexpf(E[2] - O[2], e), ldexpf(E[3] - O[3], e));
      }
    }
  }
}

// Tail differences of column c, pairs r = k0, k0 + dk, ..: rows r and C - r
// (FP64) on the end samples.  DD = d, or 0 for any d.
template <int DD>
__device__ __forceinline__ void mat_tail(const MatCtx& X, int C, int d, int c, int k0, int dk) {
  float* z = lds_f(X.z);
  if (DD) d = DD;
  for (int r = k0; r < X.Pt; r += dk) {
    const double *qa = X.dq + r * 2 * d, *qb = X.dq + (C - r) * 2 * d;
    double sa = 0.0, sb = 0.0;
#pragma unroll
    for (int j = 0; j < (DD ? DD : d); ++j) {
      const double fr = z[X.word(d - 1 - j, c) + X.hs], fl = z[X.word(j, c)];
      sa = fma(qa[j], fr, sa);
      sa = fma(qa[d + j], fl, sa);
      sb = fma(qb[j], fr, sb);
      sb = fma(qb[d + j], fl, sb);
    }
    const float xa = (float)sa, xb = r == C - r ? 0.f : (float)sb;
    float* o = z + X.word(X.Ni + r, c);
    if (r == 0 && (X.N & 1))
      X.side[c] = xa;  // the middle sample is still to be read
    else
      o[0] = xa;
    o[X.hs] = xb;
    // (the larger of |xe| and |xo|)
    atomicMax(X.cmax + c, __float_as_uint(fabsf(xa) + fabsf(xb)));
  }
}

// Derivative of every column of the tile: the samples are in LDS (stored by
// this thread block, no barrier since); on return the derivatives are in the
// samples' places, after a barrier.
template <class CLS>
__device__ __forceinline__ void mat_apply(const MatCtx& X, const PlanDev& P, const uint4* __restrict__ mt, int d) {
  const int ncp = X.ncp, ldw = X.ldw, hs = X.hs, Ni = X.Ni;
  unsigned* cm = X.cmax;
  constexpr int T = CLS::threads;
  // the thread's column, its octets of pairs k0, k0 + dk, ...
  const int tid = mat_tid(), c = tid & (ncp - 1), k0 = tid >> X.lgc, dk = T >> X.lgc;
  if (tid < ncp) cm[tid] = 0u;  // (its last readers are behind a barrier)
  __syncthreads();
  float* z = lds_f(X.z);
  // tail differences
  if (P.periodic) {
    if (k0 == 0) {  // the wrap f_0 - f_{N-1}
      const float x = z[X.word(0, c)] - z[X.word(0, c) + hs];
      float* o = z + X.word(Ni, c);
      if (X.N & 1)
        X.side[c] = x;
      else
        o[0] = x;
      o[hs] = 0.f;
      atomicMax(cm + c, __float_as_uint(fabsf(x)));
    }
  } else if (d == 5) {
    mat_tail<5>(X, P.C, d, c, k0, dk);
  } else if (d == 2) {
    mat_tail<2>(X, P.C, d, c, k0, dk);
  } else {
    mat_tail<0>(X, P.C, d, c, k0, dk);
  }
  // sums and differences of the pairs of the thread's octets, in registers,
  // and their largest
  float big = 0.f;
  float xe[CLS::items][8], xo[CLS::items][8];
  float* zc0 = z + 4 * c;                       // even rows
  float* zc1 = z + ldw + 4 * (c ^ X.odd_row(1));  // odd rows
#pragma unroll
  for (int i = 0; i < CLS::items; ++i) {
    const int k = k0 + i * dk;
    if (8 * k < Ni) {
      const int o = 2 * k * ldw;
      const int nx = k + 1 < X.KO ? o + 2 * ldw : o;  // (difference Ni - 1 is not its last)
      const float4 p = *reinterpret_cast<const float4*>(zc0 + o), p2 = *reinterpret_cast<const float4*>(zc1 + o);
      const float4 q = *reinterpret_cast<const float4*>(zc0 + o + hs),
                   q2 = *reinterpret_cast<const float4*>(zc1 + o + hs);
      float a[9] = {p.x, p.y, p.z, p.w, p2.x, p2.y, p2.z, p2.w, zc0[nx]};
      float b[9] = {q.x, q.y, q.z, q.w, q2.x, q2.y, q2.z, q2.w, zc0[nx + hs]};
      if (__builtin_amdgcn_ballot_w64((Ni - 1) >> 3 == k)) {
        // the middle of the line, difference Ni - 1.  N odd: it and its mirror
        // image share the middle sample; N even: it is its own mirror image,
        // counted once
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (8 * k + t == Ni - 1) {
            if (!(X.N & 1)) a[t + 1] = b[t];
            b[t + 1] = a[t + 1];
          }
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float xa = a[t + 1] - a[t], xb = b[t] - b[t + 1];
        xe[i][t] = xa + xb;
        xo[i][t] = xa - xb;
      }
      // (pairs from Ni on are the tail's)
      if (8 * k + 8 <= Ni) {
#pragma unroll
        for (int t = 0; t < 8; ++t) big = fmaxf(fmaxf(big, fabsf(xe[i][t])), fabsf(xo[i][t]));
      } else {
#pragma unroll
        for (int t = 0; t < 7; ++t)
          if (8 * k + t < Ni) big = fmaxf(fmaxf(big, fabsf(xe[i][t])), fabsf(xo[i][t]));
      }
    }
  }
  atomicMax(cm + c, __float_as_uint(big));
  __syncthreads();
  // the tail's pairs, scale and split in place
  const float sc = __uint_as_float((unsigned)(mat_scale(cm[c]) + 127) << 23);
#pragma unroll
  for (int i = 0; i < CLS::items; ++i) {
    const int k = k0 + i * dk;
    if (k < X.KO) {
      const int o = 2 * k * ldw;
      if (8 * k + 7 >= Ni) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int n = 8 * k + t;
          if (n >= Ni) {
            const float* s = (t < 4 ? zc0 : zc1) + o + (t & 3);
            const bool in = n < Ni + X.Pt, mid = n == Ni && (X.N & 1);
            const float xa = mid ? X.side[c] : in ? s[0] : 0.f, xb = in ? s[hs] : 0.f;
            xe[i][t] = xa + xb;
            xo[i][t] = xa - xb;
          }
        }
      }
      unsigned eh[4], el[4], oh[4], ol[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        mat_split2(xe[i][2 * t], xe[i][2 * t + 1], sc, eh[t], el[t]);
        mat_split2(xo[i][2 * t], xo[i][2 * t + 1], sc, oh[t], ol[t]);
      }
      *reinterpret_cast<uint4*>(zc0 + o) = make_uint4(eh[0], eh[1], eh[2], eh[3]);
      *reinterpret_cast<uint4*>(zc1 + o) = make_uint4(el[0], el[1], el[2], el[3]);
      *reinterpret_cast<uint4*>(zc0 + o + hs) = make_uint4(oh[0], oh[1], oh[2], oh[3]);
      *reinterpret_cast<uint4*>(zc1 + o + hs) = make_uint4(ol[0], ol[1], ol[2], ol[3]);
    }
  }
  __syncthreads();
  // one or two row blocks per wave (CLS::rows, mat_size_fits)
  constexpr int W = CLS::threads / 64, D = CLS::ahead;
  if (ncp == 16) {
    if (P.mrb <= W)
      mat_product<1, 1, D>(X, P, mt);
    else
      mat_product<2, 1, D>(X, P, mt);
  } else {
    if (P.mrb <= W)
      mat_product<1, 2, D>(X, P, mt);
    else
      mat_product<2, 2, D>(X, P, mt);
  }
  __syncthreads();
}

// Whether the kernels of a size run lines with ks K steps and rb row blocks.
template <class CLS>
inline bool mat_size_fits(int ks, int rb) {
  return 4 * ks * 32 <= CLS::items * CLS::threads && rb <= CLS::rows * (CLS::threads / 64);
}

// ---------------------------------------------------------------- tables

struct MatTab {
  int N, L, periodic, C;
  int rb, ks, es;
  long long mt;   // offset of the table in uint4
  long long kap;  // offset of kappa in doubles
};

__global__ void __launch_bounds__(256) k_mat_kappa(const MatTab* tabs, double* kap) {
  const MatTab t = tabs[blockIdx.x];
  const int L = t.L;
  const double w = t.periodic ? 2.0 * M_PI : 2.0 * M_PI * (t.N - 1) / L;
  for (int m = threadIdx.x; m < L; m += blockDim.x) {
    double s = 0.0;
    const int o = 2 * m - 1 + 2 * L;
    int ph = 0;  // k (2m - 1) mod 2L
    for (int k = 1; 2 * k < L; ++k) {
      ph = (ph + o) % (2 * L);
      s += w * k * cospi((double)ph / L) / sinpi((double)k / L);
    }
    kap[t.kap + m] = s / L;
  }
}

// One word (two halves) of a table per thread: uint4 ((rb KS + ks) 4 + 2 h +
// p) 64 + lane holds row 16 rb + lane % 16, pairs 32 ks + 8 (lane / 16) + 0..7
// of Me (h = 0) or Mo, their hi (p = 0) or lo halves.
__global__ void __launch_bounds__(256) k_mat_table(const MatTab* tabs, const double* kap, unsigned* out) {
  const MatTab t = tabs[blockIdx.y];
  const int words = t.rb * t.ks * 4 * 64 * 4;
  const int N = t.N, L = t.L, Nh = (N + 1) / 2, Ni = N / 2, Pt = (t.C + 2) / 2;
  const double* kp = kap + t.kap;
  for (int w = blockIdx.x * blockDim.x + threadIdx.x; w < words; w += gridDim.x * blockDim.x) {
    const int j = w & 3, lane = (w >> 2) & 63, p = (w >> 8) & 1, h = (w >> 9) & 1, s = w >> 10;
    const int ks = s % t.ks, i = 16 * (s / t.ks) + (lane & 15);
    unsigned word = 0;
    for (int e = 0; e < 2; ++e) {
      const int q = 32 * ks + 8 * (lane >> 4) + 2 * j + e;
      int a = -1, b = -1;
      if (q < Ni) {
        a = q;
        b = N - 2 - q;
      } else if (q < Ni + Pt) {
        a = N - 1 + (q - Ni);
        b = L - 1 - (q - Ni);
      }
      double v = 0.0;
      if (i < Nh && a >= 0) {
        const double ka = kp[(i - a + L) % L], kb = kp[(i - b + L) % L];
        v = a == b ? (h ? 0.0 : ka) : 0.5 * (h ? ka - kb : ka + kb);
      }
      v = ldexp(v, t.es);
      const _Float16 hi = (_Float16)v;
      const _Float16 x = p ? (_Float16)(v - (double)hi) : hi;
      unsigned short bits;
      __builtin_memcpy(&bits, &x, 2);
      word |= (unsigned)bits << (16 * e);
    }
    out[4 * t.mt + w] = word;
  }
}

// ---------------------------------------------------------------- passes

// Derivative along DIR of nf fields (fc_diff; pass A and the reverse mode's
// derivatives of the state), F a round.  Of one or two fields F is 2, on 16
// columns for the eight lines: on 32 they would load and multiply three or two
// copies of a field (one field along q2 of 100 patches of 128 .. 512 points 130 ->
// 107 us, of 24 patches 56 -> 46; transforms 117 and 50).
template <class CLS, int DIR, int F>
__device__ __forceinline__ void mat_diff_tile(const PassArgs& a, const TileDev& T, unsigned* lds) {
  const PlanDev P = a.plans[T.plan];
  const MatCtx X = mat_setup<F>(lds, a, P, F == 2 ? 16 : T.ld);
  const MatThread M = mat_thread<DIR>(X, P, T.nl);
  const long long base = P.off + tile_first<DIR>(T.line0, P.nb1, P.n1), pl = a.plane;
  __syncthreads();
  if constexpr (F == 2) {
    const bool two = a.nf > 1;
    const float *A = a.in + base, *B = two ? A + pl : A;
    float* z = lds_f(X.z);
    mat_walk<2 * CLS::load>(
        X, M, [&](unsigned g) { return make_float2(at(A, g), at(B, g)); },
        [&](unsigned, int w, float2 v) {
          z[w] = v.x;
          z[w + 2 * 16] = v.y;
        });
    mat_apply<CLS>(X, P, a.mt, a.d);
    float* O = a.out + base;
    mat_walk<4>(
        X, M, [](unsigned) { return 0; },
        [&](unsigned g, int w, int) {
          at(O, g) = z[w];
          if (two) at(O + pl, g) = z[w + 2 * 16];
        });
    return;
  }
  for (int f = 0; f < a.nf; f += 4) {
    const float* A = a.in + (long long)f * pl + base;
    const int n = min(4, a.nf - f);
    const long long o1 = n > 1 ? pl : 0, o2 = n > 2 ? 2 * pl : 0, o3 = n > 3 ? 3 * pl : 0;
    mat_load4<CLS>(X, M, A, A + o1, A + o2, A + o3);
    mat_apply<CLS>(X, P, a.mt, a.d);
    float* O = a.out + (long long)f * pl + base;
    const float* z = lds_f(X.z);
    const int ncp = X.ncp;
    mat_walk<4>(
        X, M, [](unsigned) { return 0; },
        [&](unsigned g, int w, int) {
          const float* p = z + w;
          at(O, g) = p[0];
          if (n > 1) at(O + pl, g) = p[ncp];
          if (n > 2) at(O + 2 * pl, g) = p[2 * ncp];
          if (n > 3) at(O + 3 * pl, g) = p[3 * ncp];
        });
    __syncthreads();
  }
}

// Passes B1 (FUSED: and B2) on a q2 tile: d2 e of the four components, H =
// mu grad_x e - f' stored, then the q2 derivatives of H two components a
// round -- components 0 and 1 from LDS, 2 and 3 read back from the H that this
// workgroup has stored (the barrier orders the stores before the loads).
template <class CLS, bool FUSED>
__device__ __forceinline__ void mat_B_tile(const PassArgs& a, const TileDev& T, unsigned* lds) {
  const PlanDev P = a.plans[T.plan];
  const MatCtx X = mat_setup(lds, a, P, T.ld);
  const MatThread M = mat_thread<2>(X, P, T.nl);
  const long long base = P.off + tile_first<2>(T.line0, P.nb1, P.n1), pl = a.plane;
  const int flux = a.mode, ncp = X.ncp;
  float* z = lds_f(X.z);
  __syncthreads();
  if (!FUSED || flux != FLUX_INVISCID) {
    const float* u = a.u + base;
    mat_load4<CLS>(X, M, u, u + pl, u + 2 * pl, u + 3 * pl);
    mat_apply<CLS>(X, P, a.mt, a.d);
  }
  const HSrc hs = h_sources(a, base, flux);
  float* H = a.H + base;
  float* d2o = a.d2out ? a.d2out + base : nullptr;
  mat_walk<CLS::epiH>(
      X, M, [&](unsigned g) { return load_H4_inputs(hs, g); },
      [&](unsigned g, int w, const HIn4& q) {
        float* p = z + w;
        float d2[4] = {p[0], p[ncp], p[2 * ncp], p[3 * ncp]};
        if (a.d2th && P.wallp) {
          // the energy's derivative by the product rule from rho, m and theta's
          // (Remark adiabatic): dE = A d rho + B d theta + (m . dm) / rho
          const float ir = 1.0f / q.e[0], mq = q.e[1] * q.e[1] + q.e[2] * q.e[2];
          const float A = q.e[3] * ir - mq * ir * ir, B = q.e[0] / (a.gamma - 1.0f);
          d2[3] = A * d2[0] + B * at(a.d2th + base, g) + (q.e[1] * d2[1] + q.e[2] * d2[2]) * ir;
        }
        if (d2o) {
#pragma unroll
          for (int k = 0; k < 4; ++k) at(d2o + k * pl, g) = d2[k];
        }
        float dF[4] = {0.f, 0.f, 0.f, 0.f}, dG[4] = {0.f, 0.f, 0.f, 0.f};
        if (flux != FLUX_VISC) dev_flux(q.e, a.eref, a.pref, a.gamma, dF, dG);
        float h[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float vx = 0.f, vy = 0.f;
          if (flux != FLUX_INVISCID) {
            vx = q.mu * (q.m1x * q.d1[k] + q.m2x * d2[k]);
            vy = q.mu * (q.m1y * q.d1[k] + q.m2y * d2[k]);
          }
          h[2 * k] = vx - dF[k];
          h[2 * k + 1] = vy - dG[k];
          at(H + (2 * k) * pl, g) = h[2 * k];
          at(H + (2 * k + 1) * pl, g) = h[2 * k + 1];
        }
        if (FUSED) {
          p[0] = h[0];
          p[ncp] = h[1];
          p[2 * ncp] = h[2];
          p[3 * ncp] = h[3];
        }
      });
  if (!FUSED) return;
  const float* m2x = a.metric + 2 * pl + base;
  const float* m2y = a.metric + 3 * pl + base;
  float* r2 = a.r2 + base;
  for (int half = 0; half < 2; ++half) {
    if (half) {
      __syncthreads();  // the first half's results have been read
      mat_load4<CLS>(X, M, H + 4 * pl, H + 5 * pl, H + 6 * pl, H + 7 * pl);
    }
    mat_apply<CLS>(X, P, a.mt, a.d);
    float* ra = r2 + (2 * half) * pl;
    mat_walk<6>(
        X, M, [&](unsigned g) { return make_float2(at(m2x, g), at(m2y, g)); },
        [&](unsigned g, int w, float2 m) {
          const float* p = z + w;
          at(ra, g) = m.x * p[0] + m.y * p[ncp];
          at(ra + pl, g) = m.x * p[2 * ncp] + m.y * p[3 * ncp];
        });
  }
}

// Pass B2 alone (split schedule): r2_c = m2x d2 H_x,c + m2y d2 H_y,c, two
// components a round.
template <class CLS>
__device__ __forceinline__ void mat_B2_tile(const PassArgs& a, const TileDev& T, unsigned* lds) {
  const PlanDev P = a.plans[T.plan];
  const MatCtx X = mat_setup(lds, a, P, T.ld);
  const MatThread M = mat_thread<2>(X, P, T.nl);
  const long long base = P.off + tile_first<2>(T.line0, P.nb1, P.n1), pl = a.plane;
  const int ncp = X.ncp;
  const float* z = lds_f(X.z);
  const float* H = a.H + base;
  const float* m2x = a.metric + 2 * pl + base;
  const float* m2y = a.metric + 3 * pl + base;
  __syncthreads();
  for (int half = 0; half < 2; ++half) {
    if (half) __syncthreads();
    const float* h = H + (4 * half) * pl;
    mat_load4<CLS>(X, M, h, h + pl, h + 2 * pl, h + 3 * pl);
    mat_apply<CLS>(X, P, a.mt, a.d);
    float* ra = a.r2 + base + (2 * half) * pl;
    mat_walk<8>(
        X, M, [&](unsigned g) { return make_float2(at(m2x, g), at(m2y, g)); },
        [&](unsigned g, int w, float2 m) {
          const float* p = z + w;
          at(ra, g) = m.x * p[0] + m.y * p[ncp];
          at(ra + pl, g) = m.x * p[2 * ncp] + m.y * p[3 * ncp];
        });
  }
}

// Pass C (q1 lines): r = m1x d1 H_x + m1y d1 H_y + r2, then store (SET / ADD)
// or the SSPRK register update (RK); two components a round.
template <class CLS>
__device__ __forceinline__ void mat_C_tile(const PassArgs& a, const TileDev& T, unsigned* lds) {
  const PlanDev P = a.plans[T.plan];
  const MatCtx X = mat_setup(lds, a, P, T.ld);
  const MatThread M = mat_thread<1>(X, P, T.nl);
  const long long base = P.off + tile_first<1>(T.line0, P.nb1, P.n1), pl = a.plane;
  const int ncp = X.ncp;
  const float* z = lds_f(X.z);
  const RkCoef K = rk_coef(a.stage);
  const bool rk = a.mode == MODE_RK;
  const float dt = rk ? a.dt[0] : 0.f;
  const float* m1x = a.metric + base;
  const float* m1y = a.metric + pl + base;
  __syncthreads();
  for (int half = 0; half < 2; ++half) {
    if (half) __syncthreads();
    const float* h = a.H + (4 * half) * pl + base;
    mat_load4<CLS>(X, M, h, h + pl, h + 2 * pl, h + 3 * pl);
    mat_apply<CLS>(X, P, a.mt, a.d);
    const long long fo = (2 * half) * pl + base;
    // point inputs: the q1 metric row, r2 and the SSPRK registers of the
    // stage; every load is issued (registers the stage does not use read r2)
    const float* r2c = a.r2 + fo;
    const float* uic = rk ? a.ui + fo : r2c;
    const float* wc = a.mode == MODE_ADD ? a.rhs + fo : ((rk && a.stage >= 3) ? a.acc + fo : r2c);
    const float* u0c = (rk && a.stage <= 3) ? a.u0 + fo : r2c;
    float* rhs = a.rhs + fo;
    float* uout = a.uout + fo;
    float* acc = a.acc + fo;
    struct CIn {
      float m1x, m1y, r2[2], ui[2], w[2], u0[2];
    };
    mat_walk<CLS::epiC>(
        X, M,
        [&](unsigned g) {
          CIn q;
          q.m1x = at(m1x, g);
          q.m1y = at(m1y, g);
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            q.r2[k] = at(r2c + k * pl, g);
            q.ui[k] = at(uic + k * pl, g);
            q.w[k] = at(wc + k * pl, g);
            q.u0[k] = at(u0c + k * pl, g);
          }
          return q;
        },
        [&](unsigned g, int w, const CIn& q) {
          const float* p = z + w;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const float r = q.m1x * p[(2 * k) * ncp] + q.m1y * p[(2 * k + 1) * ncp] + q.r2[k];
            if (a.mode == MODE_SET) {
              at(rhs + k * pl, g) = r;
            } else if (a.mode == MODE_ADD) {
              at(rhs + k * pl, g) = q.w[k] + r;
            } else {
              const float ui = q.ui[k], dr = dt * r;
              if (a.stage <= 3)
                at(uout + k * pl, g) = K.a0 * q.u0[k] + K.ai * ui + K.b * dr;
              else
                at(uout + k * pl, g) = q.w[k] + K.ai * ui + K.b * dr;
              if (a.stage == 2) at(acc + k * pl, g) = K.acc_i * ui;
              if (a.stage == 3) at(acc + k * pl, g) = q.w[k] + (K.acc_i * ui + K.acc_b * dr);
            }
          }
        });
  }
}

#define FCSD_MAT_KERNEL(call)                    \
  const TileDev T = a.tiles[blockIdx.x];         \
  if (T.nl == 0) return;                         \
  unsigned* lds = reinterpret_cast<unsigned*>(lds_z); \
  call(a, T, lds);

template <class CLS, int DIR, int F>
__global__ void FCSD_MAT_BOUNDS(CLS) k_mat_diff(PassArgs a) {
  FCSD_MAT_KERNEL((mat_diff_tile<CLS, DIR, F>))
}
template <class CLS, bool FUSED>
__global__ void FCSD_MAT_BOUNDS(CLS) k_mat_B(PassArgs a) {
  FCSD_MAT_KERNEL((mat_B_tile<CLS, FUSED>))
}
template <class CLS>
__global__ void FCSD_MAT_BOUNDS(CLS) k_mat_B2(PassArgs a) {
  FCSD_MAT_KERNEL(mat_B2_tile<CLS>)
}
template <class CLS>
__global__ void FCSD_MAT_BOUNDS(CLS) k_mat_C(PassArgs a) {
  FCSD_MAT_KERNEL(mat_C_tile<CLS>)
}

// ---------------------------------------------------------------- one launch per stage

// Task kinds of the persistent stage kernel: pass A on a q1 tile, passes
// B1 + B2 on a q2 tile, pass C on a q1 tile; TASK_MAT: a tile of lines that
// run as matrix products.
enum { TASK_A = 0, TASK_B = 1, TASK_C = 2, TASK_MAT = 4 };

struct StageArgs {
  PassArgs A, B, C;         // the passes' arguments
  const TileDev *q1[2], *q2[2];  // tiles of the lines that run as transforms, as products
  const int2* tasks;        // (kind, tile index), in queue order
  int ntasks;
  int npatch;
  int skipA;                // inviscid stage: A tasks do nothing
  unsigned* ctr;            // [0] queue head; [1 + p] A tiles done of patch p; [1 + np + p] B tiles done
  const unsigned* need;     // [p] A tiles of patch p; [np + p] B tiles of patch p
  unsigned* err;            // bit 0 set when a wait gave up (results of the launch are then invalid)
};

// Upper bound on the polls of one dependency wait (each poll sleeps ~128
// cycles: about a second in all), after which the workgroup records the
// failure in err and goes on, so that every workgroup ends.
constexpr int kSpinLimit = 1 << 24;

// One RK stage in one launch: every workgroup takes tasks from a global
// queue until it is empty.  The queue holds all A tasks, then every B task,
// then every C task, so a task only depends on tasks taken before it (B on
// its patch's A tiles, C on its patch's B tiles), which are held by running
// workgroups: the earliest unfinished task can always proceed, whatever the
// number of resident workgroups.  A task's completion is published by a
// release increment of its patch's counter after a workgroup barrier (every
// thread's stores are then complete); a dependent task starts after an
// acquire poll of that counter.  Phases of different patches overlap, and no
// workgroup idles at the end of a pass.  The counters start at zero (the
// host clears them before the launch).  FFT, MAT: the queue holds tiles of
// transforms, of products.
template <bool FFT, bool MAT>
__device__ __forceinline__ void stage_tasks(const StageArgs& s) {
  // the first 16 bytes of the dynamic LDS hold the task index; tiles start after
  int* slot = reinterpret_cast<int*>(lds_z);
  float2* lds = lds_z + 2;
  unsigned* mlds = reinterpret_cast<unsigned*>(lds);
  const int np = s.npatch;
  for (;;) {
    __syncthreads();  // the previous task's LDS reads are done; the slot is free
    if (threadIdx.x == 0) slot[0] = (int)atomicAdd(s.ctr, 1u);
    __syncthreads();
    const int t = slot[0];
    if (t >= s.ntasks) return;
    const int2 k = s.tasks[t];
    const int kind = k.x & 3;
    const bool mat = MAT && (!FFT || (k.x & TASK_MAT));
    const TileDev T = (kind == TASK_B ? s.q2 : s.q1)[mat][k.y];
    const int p = T.plan;  // one plan per patch and direction
    if (kind != TASK_A) {
      if (threadIdx.x == 0) {
        const int dep = (kind == TASK_B ? 0 : np) + p;
        const unsigned need = s.need[dep];
        unsigned* c = s.ctr + 1 + dep;
        int polls = 0;
        while (__hip_atomic_load(c, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < need) {
          if (++polls > kSpinLimit) {
            atomicOr(s.err, 1u);
            break;
          }
          __builtin_amdgcn_s_sleep(2);
        }
      }
      __syncthreads();
    }
    if constexpr (MAT) {
      if (mat) {
        if (kind == TASK_A) {
          if (!s.skipA) mat_diff_tile<MatLarge, 1, 4>(s.A, T, mlds);
        } else if (kind == TASK_B) {
          mat_B_tile<MatLarge, true>(s.B, T, mlds);
        } else {
          mat_C_tile<MatLarge>(s.C, T, mlds);
        }
      }
    }
    if constexpr (FFT) {
      if (!mat) {
        if (kind == TASK_A) {
          if (!s.skipA) dev_diff_tile<1>(s.A, T, lds);
        } else if (kind == TASK_B) {
          passB_tile<true>(s.B, T, lds);
        } else {
          passC_tile(s.C, T, lds);
        }
      }
    }
    if (kind != TASK_C) {
      __syncthreads();  // every thread's stores of the task are complete
      if (threadIdx.x == 0)
        __hip_atomic_fetch_add(s.ctr + 1 + (kind == TASK_A ? 0 : np) + p, 1u, __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

__global__ void FCSD_LINE_BOUNDS k_stage(StageArgs s) { stage_tasks<true, false>(s); }

// Sets with products: the products' workgroup size for every task.
template <bool FFT>
__global__ void FCSD_MAT_BOUNDS(MatLarge) k_stage_mat(StageArgs s) {
  stage_tasks<FFT, true>(s);
}

}  // namespace fcsd
