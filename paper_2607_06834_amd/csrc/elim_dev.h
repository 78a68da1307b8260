// X = L^-1 of a symmetric positive-definite matrix A = L L^T of T x T tiles of
// 16 x 16, by block Gauss-Jordan elimination with the tiles held in registers.
//
// W waves work on a problem.  The T (T + 1) / 2 lower tiles (I, C), C <= I, are
// dealt to them in order: wave w holds the tiles s W + w in its slots s.  At
// step J the slot of tile (I, C) holds
//   C >= J:       -A_CI (rows of block C, columns of block I; A is symmetric),
//   C < J <= I:   -Y_IC, the block column C of L^-1 as far as it is formed,
//   I < J:        X_IC, final,
// so that a slot is never idle storage and the matrix needs no memory of its
// own.  Step J:
//   1. the wave that holds (J, J) factorises it and inverts the factor: X_JJ
//      to LDS (with several waves one step ahead, right after that tile's
//      update);
//   2. the tiles of row J: R_JI = X_JJ A_JI (= L_IJ^T, I > J) and
//      X_JC = X_JJ Y_JC (C < J), to the LDS row buffer;
//   3. every other tile below row J takes one product of two tiles of that row,
//      -A_CI += R_JC^T R_JI, -Y_IC += R_JI^T X_JC, and -Y_IJ = R_JI^T X_JJ.
// Every operand of step 3 is a tile of the row buffer as it was written (the
// transposed one is the A operand of the matrix instruction, see below), the
// accumulator stays in its slot and is never negated, and there are two
// barriers a step.
//
// Layout of a tile held by a wave (lane l = c + 16 q): element v is
// M[q + 4 v][c], the result layout of v_mfma_f64_16x16x4f64 and its B operand;
// the same registers are the A operand of M^T.  In v_mfma_f64_4x4x4f64 (four
// blocks of four columns) one of these registers is the B operand too, and with
// A[i][k] = y_i[k] the result is sum_k y_i[4 v + k] M[4 v + k][c] in lane
// c + 16 i: products M^T y of up to four vectors with no exchange between lanes.
//
// LDS tiles have rows of 17 doubles: both a tile's rows and its columns are read
// by 16 lanes from different banks, with the four elements of a lane at fixed
// offsets.  Vectors come in pairs, [row][2].
#pragma once

#include <cmath>

#include "lane_dev.h"
#include "std.h"

namespace el {

using ln::v4d;

constexpr int kLd = 17, kTile = 16 * kLd;

__device__ inline v4d ld_rm(const double *t, int c, int q) {   // M[c][q + 4s]: A operand of M
  const double *p = t + c * kLd + q;
  return v4d{p[0], p[4], p[8], p[12]};
}
__device__ inline v4d ld_cm(const double *t, int c, int q) {   // M[q + 4v][c]: B operand, A operand of M^T
  const double *p = t + q * kLd + c;
  return v4d{p[0], p[4 * kLd], p[8 * kLd], p[12 * kLd]};
}
__device__ inline void st_cm(double *t, int c, int q, v4d v) {
  double *p = t + q * kLd + c;
  p[0] = v[0];
  p[4 * kLd] = v[1];
  p[8 * kLd] = v[2];
  p[12 * kLd] = v[3];
}
// rows 4v + q of a pair of vectors y ([16][2]): the A operand of pair_tdot
__device__ inline v4d ld_pair(const double *y, int c, int q) {
  const double *p = y + 2 * q + (c & 1);
  return v4d{p[0], p[8], p[16], p[24]};
}
// M^T y for the pair of vectors y: entry c of vector i in the lanes c + 16 i,
// i = 0, 1 (and again in i + 2)
__device__ inline double pair_tdot(const v4d &y, const v4d &m) {
  double s = __builtin_amdgcn_mfma_f64_4x4x4f64(y[0], m[0], 0.0, 0, 0, 0);
  s = __builtin_amdgcn_mfma_f64_4x4x4f64(y[1], m[1], s, 0, 0, 0);
  s = __builtin_amdgcn_mfma_f64_4x4x4f64(y[2], m[2], s, 0, 0, 0);
  return __builtin_amdgcn_mfma_f64_4x4x4f64(y[3], m[3], s, 0, 0, 0);
}

// 1 / a and 1 / sqrt(a) from the hardware estimates (relative error below
// 2^-22) by one third-order step: the remaining error, of the cube of the
// estimate's, is below that of the last rounding.  The pivot chain waits on
// the reciprocal, and this is three dependent operations instead of four.
__device__ inline double rcp_c(double a) {
  const double y = __builtin_amdgcn_rcp(a);
  const double e = fma(-a, y, 1.0);
  return fma(y, fma(e, e, e), y);
}
__device__ inline double rsqrt_c(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  const double e = fma(-a * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// The symmetric tile A (all of it), given as n = -A -> X = L^-1 (zeros above the
// diagonal), A = L L^T; one wave.  Four pivots at a time: register b of the tile
// is the strip of rows 4b .. 4b + 3, row q in lane row q.  The strip's 4 x 4 block
// goes to every lane through LDS (scr, 64 doubles) and is factorised and
// inverted there (l_4^-1, no further exchange between lanes); one 4x4x4 matrix
// instruction applies l_4^-1 to the strip of A and one to the strip of the
// identity that becomes X, and one 16x16x4 instruction each updates the rows
// below.  The instructions issued set the time of a lone wave: 16 pivots one by
// one, each with its row broadcast to the lane rows, took 60 instructions and
// 310 cycles a pivot, 5.0e3 cycles a tile.
// rs[j] (LDS) receives 1 / L_jj = X_jj.  With LZ, the pair lzd[c] = (L tz)_c
// (LDS).  r receives L^T.  ok is cleared in the lanes that see a pivot that is
// not positive and finite.
template <bool LZ>
__device__ __forceinline__ v4d diag(v4d n, bool &ok, int c, int q, double *scr, double *rs, const double *tz,
                                    double *lzd, v4d &r) {
  // opaque to the compiler, which would otherwise keep the lane masks below in
  // scalar registers across the caller's loop (and spill them)
  asm volatile("" : "+v"(c), "+v"(q));
  constexpr int kPositive = 0x100 | 0x80;   // class: normal or denormal above zero
  v4d e;                                    // minus the identity, then X strip by strip
#pragma unroll
  for (int v = 0; v < 4; ++v) e[v] = (q + 4 * v == c) ? -1.0 : 0.0;
  const int i = c & 3;
  double part = 0.0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    double s = n[b], f = e[b];
    scr[16 * q + c] = s;
    const double2 *m = reinterpret_cast<const double2 *>(scr) + 2 * b;   // minus the block, two by two
    const double2 r0 = m[0], r1 = m[8], r2 = m[16], r3 = m[24], r2b = m[17], r3b = m[25];
    // l_4 D l_4^T of the block, then the inverse of the unit lower l_4
    const double i0 = rcp_c(-r0.x);
    const double l10 = -r1.x * i0, l20 = -r2.x * i0, l30 = -r3.x * i0;
    const double d1 = fma(l10, r1.x, -r1.y), m21 = fma(l20, r1.x, -r2.y), m31 = fma(l30, r1.x, -r3.y);
    const double i1 = rcp_c(d1);
    const double l21 = m21 * i1, l31 = m31 * i1;
    const double d2 = fma(-l21, m21, fma(l20, r2.x, -r2b.x));
    const double m32 = fma(-l31, m21, fma(l30, r2.x, -r3b.x));
    const double i2 = rcp_c(d2);
    const double l32 = m32 * i2;
    const double d3 = fma(-l32, m32, fma(-l31, m31, fma(l30, r3.x, -r3b.y)));
    // minus the inverse u of l_4
    const double u20 = fma(-l21, l10, l20), u31 = fma(-l32, l21, l31);
    const double u30 = fma(-l32, u20, fma(-l31, l10, l30));
    // element (i, q) of -l_4^-1 = -D^-1/2 u, i = c mod 4: the A operand
    const double di = (i & 2) ? ((i & 1) ? d3 : d2) : ((i & 1) ? d1 : -r0.x);
    ok = ok && __builtin_amdgcn_class(di, kPositive);
    const double ri = rsqrt_c(di);
    double u = (q == i) ? -1.0 : 0.0;
    u = (q == 0 && i == 1) ? l10 : u;
    u = (q == 0 && i == 2) ? u20 : u;
    u = (q == 0 && i == 3) ? u30 : u;
    u = (q == 1 && i == 2) ? l21 : u;
    u = (q == 1 && i == 3) ? u31 : u;
    u = (q == 2 && i == 3) ? l32 : u;
    u *= ri;
    s = __builtin_amdgcn_mfma_f64_4x4x4f64(u, s, 0.0, 0, 0, 0);
    f = __builtin_amdgcn_mfma_f64_4x4x4f64(u, f, 0.0, 0, 0, 0);
    e[b] = f;
    if (q == 0 && c < 4) rs[4 * b + c] = ri;
    r[b] = c >= 4 * b + q ? s : 0.0;
    if (LZ) part = __builtin_amdgcn_mfma_f64_4x4x4f64(tz[2 * (4 * b + q) + (c & 1)], r[b], part, 0, 0, 0);
    if (b < 3) {
      const double sm = (c >= 4 * b + 4) ? s : 0.0;   // the rows below the strip
      n = __builtin_amdgcn_mfma_f64_16x16x4f64(sm, s, n, 0, 0, 0);
      e = __builtin_amdgcn_mfma_f64_16x16x4f64(sm, f, e, 0, 0, 0);
    }
  }
  if (LZ && q < 2) lzd[2 * c + q] = part;
  return e;
}

// LDS of an elimination: the row buffer, X_JJ (two buffers where it is formed a
// step ahead), and the diagonal work.
template <int T, int W>
struct Lds {
  double row[T * kTile];
  double xd[(W > 1 ? 2 : 1) * kTile];
  double scr[64];
  double rs[16 * T];    // 1 / L_jj
  double lzd[32 * T];   // the diagonal tiles' part of L z
  __device__ inline double *xjj(int J) { return xd + (W > 1 ? (J & 1) * kTile : 0); }
};

struct NoSink {
  static constexpr bool kOn = false;
};

template <int T, int W>
struct Elim {
  static constexpr int NT = ps::ntiles(T), NS = (NT + W - 1) / W;
  static_assert(NS <= 16, "tile indices in nibbles");
  int w, lane, c, q;
  uint64_t ti, tc;   // the tile (I, C) of each slot, in nibbles
  v4d a[NS];

  __device__ __forceinline__ explicit Elim(int tid)
      : w(W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6)), lane(tid & 63), c(tid & 15), q((tid & 63) >> 4),
        ti(0), tc(0) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int t = s * W + w;
      int i = 0;
#pragma unroll
      for (int k = 1; k < T; ++k) i += t >= ps::tix(k, 0);
      ti |= (uint64_t)(t < NT ? i : 0) << (4 * s);
      tc |= (uint64_t)(t < NT ? t - ps::tix(i, 0) : 0) << (4 * s);
    }
  }
  __device__ __forceinline__ int tile_i(int s) const { return (int)(ti >> (4 * s)) & 15; }
  __device__ __forceinline__ int tile_c(int s) const { return (int)(tc >> (4 * s)) & 15; }
  __device__ __forceinline__ bool has(int s) const { return (s + 1) * W <= NT || s * W + w < NT; }

  // factor and inverse of the diagonal tile n = -A_JJ; X_JJ to LDS
  template <bool LZ, class Sink>
  __device__ __forceinline__ v4d pivot(const v4d &n, int J, Lds<T, W> &L, int *flag, const double *tv, Sink &sink) {
    bool ok = true;
    v4d r;
    const v4d x = diag<LZ>(n, ok, c, q, L.scr, L.rs + 16 * J, LZ ? tv + 32 * J : nullptr, L.lzd + 32 * J, r);
    st_cm(L.xjj(J), c, q, x);
    if constexpr (Sink::kOn) sink.diagonal(J, r);
    if (!__all(ok) && lane == 0) *flag = 0;
    return x;
  }

  // The whole elimination of the slots' -A.  Of the pairs bv and tv ([16 T][2],
  // LDS) the first NB are right-hand sides b (consumed) and t = X b; the next
  // NZ of tv are vectors z, and L z is theirs of bv (zero on entry) plus L.lzd.
  // hook(J) runs in step 3, when row J of X is complete (X_JC, C < J, at
  // L.row + kTile C, X_JJ at L.xjj(J)).  A sink takes the factor: diagonal(J,
  // L_JJ^T) and below(I, J, rows q + 4 v of L_IJ).  INV false leaves X out (the
  // factor, t and L z only).  flag (LDS) is cleared when a pivot fails.  All
  // 64 W threads call it, after a barrier that follows the caller's writes of
  // bv, tv and flag.
  template <int NB, int NZ, bool INV = true, class Hook, class Sink = NoSink>
  __device__ __forceinline__ void run(Lds<T, W> &L, int *flag, double *bv, double *tv, Hook hook, Sink sink = Sink()) {
    if (w == 0) a[0] = pivot<(NZ > 0)>(a[0], 0, L, flag, tv, sink);
    __syncthreads();
    if constexpr (W == 1 && T <= 4) {   // one wave: the tiles of each step are known
#pragma unroll
      for (int J = 0; J < T; ++J) step<NB, NZ, INV>(J, L, flag, bv, tv, hook, sink);
    } else {
#pragma unroll 1
      for (int J = 0; J < T; ++J) {
        // opaque in the loop, so that the addresses formed from the tiles are
        // not kept in registers across it
        if (W > 1) asm volatile("" : "+s"(ti), "+s"(tc));
        step<NB, NZ, INV>(J, L, flag, bv, tv, hook, sink);
      }
    }
  }

  template <int NB, int NZ, bool INV, class Hook, class Sink>
  __device__ __forceinline__ void step(int J, Lds<T, W> &L, int *flag, double *bv, double *tv, Hook &hook, Sink &sink) {
    static_assert(NB + NZ <= 2, "one pair of vectors");
    constexpr bool kVec = NB + NZ > 0, LZ = NZ > 0;
    double *xj = L.xjj(J);
    // 2. row J
    {
      const v4d xa = ld_rm(xj, c, q), xn = -xa;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int I = tile_i(s), C = tile_c(s);
        if ((INV ? (I == J) != (C == J) : (I != J && C == J)) && has(s)) {
          const v4d r = ln::mfma4(xn, a[s], v4d{0.0, 0.0, 0.0, 0.0});
          st_cm(L.row + kTile * (I == J ? C : I), c, q, r);
          if constexpr (Sink::kOn)
            if (C == J) sink.below(I, J, ld_rm(L.row + kTile * I, c, q));
          a[s] = r;
          if (C == J) a[s] = v4d{0.0, 0.0, 0.0, 0.0};   // Y_IJ starts in step 3
        }
      }
      if (NB > 0 && w == J % W) {
        const double t = pair_tdot(ld_pair(bv + 32 * J, c, q), xa);
        if (q < NB) tv[2 * (16 * J + c) + q] = t;
      }
    }
    __syncthreads();
    // 3. with several waves the next diagonal tile first, ahead of the other
    // waves of the compute unit: the step waits for it
    const bool own = W > 1 && J + 1 < T && w == ps::tix(J + 1, J + 1) % W;
    const int sd = own ? ps::tix(J + 1, J + 1) / W : -1;
    if (own) {
      __builtin_amdgcn_s_setprio(2);
      v4d d;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s == sd) d = a[s];
      const v4d r = ld_cm(L.row + kTile * (J + 1), c, q);
      const v4d x = pivot<LZ>(ln::mfma4(r, r, d), J + 1, L, flag, tv, sink);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s == sd) a[s] = x;
      __builtin_amdgcn_s_setprio(0);
    }
    hook(J);
    v4d ty;
    if (kVec) ty = ld_pair(tv + 32 * J, c, q);
    // the slots from the last (tiles are dealt by rows: the first one at or
    // above row J ends the loop), the next slot's operands loaded ahead
    v4d u, v;
    operands(NS - 1, J, L, xj, u, v);
#pragma unroll
    for (int s = NS - 1; s >= 0; --s) {
      v4d un{}, vn{};
      if (has(s)) {
        if (tile_i(s) <= J) break;
        if (s > 0) operands(s - 1, J, L, xj, un, vn);
        if (s != sd) {
          if (INV || tile_c(s) > J) a[s] = ln::mfma4(u, v, a[s]);
          if (kVec && tile_c(s) == J) {   // b -= R_JI^T t, L z += R_JI^T z
            const double e = pair_tdot(ty, u);
            if (q < NB + NZ) {
              double *o = bv + 2 * (16 * tile_i(s) + c) + q;
              *o = q < NB ? *o - e : *o + e;
            }
          }
        }
      } else {
        operands(s - 1, J, L, xj, un, vn);
      }
      u = un;
      v = vn;
    }
    if (W == 1 && J + 1 < T) {
      const int s1 = ps::tix(J + 1, J + 1);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s == s1) a[s] = pivot<LZ>(a[s], J + 1, L, flag, tv, sink);
    }
    __syncthreads();
  }

  // The tiles of row J that update slot s: R_JC, R_JI while the slot holds A, and
  // R_JI, X_JC after.  Any slot gives addresses within the buffers.
  __device__ __forceinline__ void operands(int s, int J, const Lds<T, W> &L, const double *xj, v4d &u, v4d &v) const {
    const int I = tile_i(s), C = tile_c(s);
    const bool tr = C > J;
    u = ld_cm(L.row + kTile * (tr ? C : I), c, q);
    v = ld_cm(C == J ? xj : L.row + kTile * (tr ? I : C), c, q);
  }

  // Column sums X^T y of the pair y ([16 T][2], LDS) over the wave's tiles, tile
  // by tile to part[tix(I, C)][2][16] (LDS); after a barrier xty_sum adds a
  // column's tiles in order.
  __device__ __forceinline__ void xty(double *part, const double *y) const {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (!has(s)) continue;
      const double u = pair_tdot(ld_pair(y + 32 * tile_i(s), c, q), a[s]);
      if (q < 2) part[(s * W + w) * 32 + 16 * q + c] = u;
    }
  }
  // the squared columns of X likewise, to part[tix(I, C)][16]
  __device__ __forceinline__ void xsq(double *part) const {
    const v4d one{1.0, 1.0, 1.0, 1.0};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (!has(s)) continue;
      const double u = pair_tdot(one, a[s] * a[s]);
      if (q == 0) part[(s * W + w) * 16 + c] = u;
    }
  }
};

// entry r of a column sum from its tiles' parts, N values of 16 columns a tile
template <int T, int N>
__device__ inline double xty_sum(const double *part, int k, int r) {
  double s = 0.0;
  for (int I = r >> 4; I < T; ++I) s += part[(ps::tix(I, r >> 4) * N + k) * 16 + (r & 15)];
  return s;
}

// X for the adjoint: block columns one after the other, the rows 16 C .. 16 T - 1
// of block column C as [row][16].  cix: first row of a block column in it.
template <int T>
__host__ __device__ constexpr int cix(int C) { return 16 * (C * T - C * (C - 1) / 2); }

template <int T, int W>
__device__ __forceinline__ void store_x(const Elim<T, W> &E, double *__restrict__ xo) {
#pragma unroll
  for (int s = 0; s < Elim<T, W>::NS; ++s) {
    if (!E.has(s)) continue;
    const int I = E.tile_i(s), C = E.tile_c(s);
    double *o = xo + (cix<T>(C) + 16 * (I - C)) * 16 + 16 * E.q + E.c;
#pragma unroll
    for (int v = 0; v < 4; ++v) o[64 * v] = E.a[s][v];
  }
}

}  // namespace el
