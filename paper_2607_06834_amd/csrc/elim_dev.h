// X = L^-1 of a symmetric positive-definite matrix A = L L^T of T x T tiles of
// 16 x 16, by block Gauss-Jordan elimination with the tiles held in registers.
//
// One wave works on a problem, or W = 4 of which three hold the tiles and one
// does the diagonal tiles.  Of the T (T + 1) / 2 lower tiles (I, C), C <= I, wave
// w of the three holds those of (I + C) mod 3 = w in its slots, row by row (each
// row and each column is spread evenly).  At step J the slot of tile (I, C) holds
//   C >= J:       -A_CI (rows of block C, columns of block I; A is symmetric),
//   C < J <= I:   -Y_IC, the block column C of L^-1 as far as it is formed,
//   I < J:        X_IC, final,
// so that a slot is never idle storage and the matrix needs no memory of its
// own.  Step J:
//   1. (J, J) is factorised and its factor inverted, X_JJ to LDS: by the wave
//      itself, or by the fourth one a step ahead, beside steps 2 and 3 of J - 1.
//      It forms that step's R and its update of the tile itself, from the tiles
//      (J, J - 1) and (J, J) as of step J - 2, which their holders left in LDS,
//      and does the first four pivots before the barrier between 2 and 3;
//   2. the tiles of row J: R_JI = X_JJ A_JI (= L_IJ^T, I > J) and
//      X_JC = X_JJ Y_JC (C < J), to the LDS row buffer;
//   3. every other tile below row J takes one product of two tiles of that row,
//      -A_CI += R_JC^T R_JI, -Y_IC += R_JI^T X_JC, and -Y_IJ = R_JI^T X_JJ.
// Every operand of step 3 is a tile of the row buffer as it was written (the
// transposed one is the A operand of the matrix instruction, see below), the
// accumulator stays in its slot and is never negated, and there are two
// barriers a step.
//
// Why a wave of its own, and always on the same SIMD (placed_tid), for the
// diagonal tiles: their 16 pivots are about 170 dependent FP64 vector operations
// and 700 instructions, 3.5e3 cycles in a wave alone, and every step waits for
// them.  An FP64 operation waits for the matrix instruction that another wave of
// its SIMD has in the FP64 unit, up to 64 cycles, so among the products of three
// problems a compute unit the pivots took 10e3 to 15e3.  The fourth SIMD's share
// of the products (57e3 cycles a problem at T = 8) goes to the other three, and
// the diagonal tiles of several problems overlap on it.  T = 8, 4288 problems:
// four waves that hold nine tiles each and take turns with the diagonal 297 us,
// as here 236 (a problem alone: 48e3 cycles, of which steps 2 and 3 take 34e3 in
// either kind of wave; three problems a compute unit: 71e3; the products' share
// of the three SIMDs is 53 %).  What bounds it: the rate at which a SIMD issues
// for the three waves on it, and the 25 % of a problem's time before its first
// and after its last step.
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
// -t by the sign bits (the FP64 unit is not needed)
__device__ inline double neg(double v) { return __hiloint2double(__double2hiint(v) ^ (int)0x80000000, __double2loint(v)); }
__device__ inline v4d neg(const v4d &t) { return v4d{neg(t[0]), neg(t[1]), neg(t[2]), neg(t[3])}; }
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
// 2^-24) by one third-order step: the remaining error, of the cube of the
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
// rs[j] (LDS) receives 1 / L_jj = X_jj.  With LZ, part is (L tz)_c of vector q.
// After the strips 0 .. 3, e is X and r is L^T.  ok is cleared in the lanes that
// see a pivot that is not positive and finite.
template <bool LZ>
struct Diag {
  v4d n, e, r;     // -A, minus the identity and then X strip by strip, L^T
  double h[4];     // minus column q of the 4 x 4 identity
  double part;
  int c, q;
  bool ok;

  __device__ __forceinline__ Diag(const v4d &n_, int c_, int q_) : n(n_), part(0.0), c(c_), q(q_), ok(true) {
    // opaque to the compiler, which would otherwise keep the lane masks below in
    // scalar registers across the caller's loop (and spill them)
    asm volatile("" : "+v"(c), "+v"(q));
#pragma unroll
    for (int v = 0; v < 4; ++v) e[v] = (q + 4 * v == c) ? -1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) h[k] = (q == k) ? -1.0 : 0.0;
  }

  template <int b>
  __device__ __forceinline__ void strip(double *scr, double *rs, const double *tz) {
    constexpr int kPositive = 0x100 | 0x80;   // class: normal or denormal above zero
    const bool o1 = c & 1, o2 = c & 2;        // i = c mod 4
    double s = n[b], f = e[b];
    if (b > 0) ln::wave_sync();   // the strip before has read its block
    scr[16 * q + c] = s;
    ln::wave_sync();
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
    double d3 = fma(-l32, m32, fma(-l31, m31, fma(l30, r3.x, -r3b.y)));
    // opaque, or the compiler moves it and its LDS read into a branch of the lanes
    asm volatile("" : "+v"(d3));
    // minus column q of the inverse of l_4; element i of it, scaled by D^-1/2, is
    // the A operand
    const double x1 = fma(-l10, h[0], h[1]);
    const double x2 = fma(-l21, x1, fma(-l20, h[0], h[2]));
    const double x3 = fma(-l32, x2, fma(-l31, x1, fma(-l30, h[0], h[3])));
    const double di = o2 ? (o1 ? d3 : d2) : (o1 ? d1 : -r0.x);
    ok = ok && __builtin_amdgcn_class(di, kPositive);
    const double ri = rsqrt_c(di);
    const double u = (o2 ? (o1 ? x3 : x2) : (o1 ? x1 : h[0])) * ri;
    s = __builtin_amdgcn_mfma_f64_4x4x4f64(u, s, 0.0, 0, 0, 0);
    f = __builtin_amdgcn_mfma_f64_4x4x4f64(u, f, 0.0, 0, 0, 0);
    e[b] = f;
    rs[4 * b + (c & 3)] = ri;   // (the same value from sixteen lanes)
    r[b] = c >= 4 * b + q ? s : 0.0;
    if (LZ) part = __builtin_amdgcn_mfma_f64_4x4x4f64(tz[2 * (4 * b + q) + (c & 1)], r[b], part, 0, 0, 0);
    if (b < 3) {
      const double sm = (c >= 4 * b + 4) ? s : 0.0;   // the rows below the strip
      n = __builtin_amdgcn_mfma_f64_16x16x4f64(sm, s, n, 0, 0, 0);
      e = __builtin_amdgcn_mfma_f64_16x16x4f64(sm, f, e, 0, 0, 0);
    }
  }
};

// LDS of an elimination: the row buffer, X_JJ (two buffers where it is formed a
// step ahead), and the diagonal work.
template <int T, int W>
struct Lds {
  double row[T * kTile];
  double xd[(W > 1 ? 2 : 1) * kTile];
  double dg[W > 1 ? 2 * kTile : 2];   // tiles (J + 1, J + 1) and (J + 1, J) as of step J - 1
  alignas(16) double scr[64];
  double rs[16 * T];    // 1 / L_jj
  double lzd[32 * T];   // the diagonal tiles' part of L z
  __device__ inline double *xjj(int J) { return xd + (W > 1 ? (J & 1) * kTile : 0); }
};

struct NoSink {
  static constexpr bool kOn = false;
};

// Thread index of a workgroup of W = 4 waves numbered by the SIMD they run on, so
// that wave 3 of every workgroup is on the same one (the four waves of a
// workgroup are placed on the four SIMDs in turn, from any of them); numbered as
// launched if two waves share a SIMD.  Which SIMD the first wave gets differs from
// workgroup to workgroup, so whatever is shared among the waves and put together
// again goes by this index, not by threadIdx.x: then only which wave does what
// depends on the placement.  Has a barrier; all threads call it.
template <int W>
__device__ __forceinline__ int placed_tid() {
  static_assert(W == 1 || W == 4, "one wave or one per SIMD");
  if constexpr (W == 1) {
    return threadIdx.x;
  } else {
    __shared__ int simd[W];
    constexpr int kHwId = 4, kSimdBits = (1 << 11) | (4 << 6);   // two bits from bit 4
    const int me = (int)__builtin_amdgcn_s_getreg(kSimdBits | kHwId) & 3;
    if ((threadIdx.x & 63) == 0) simd[threadIdx.x >> 6] = me;
    __syncthreads();
    const int seen = 1 << simd[0] | 1 << simd[1] | 1 << simd[2] | 1 << simd[3];
    return seen == 15 ? 64 * me + (threadIdx.x & 63) : threadIdx.x;
  }
}

// The tiles of each tile-holding wave: their rows and columns in nibbles, and for
// each step the slots with a tile in its row or column, 16 bits a step.
template <int T, int NW>
struct Deal {
  uint64_t ti[NW], tc[NW], rows[NW][2];
  int n[NW], most, least;
  constexpr Deal() : ti{}, tc{}, rows{}, n{}, most(0), least(0) {
    for (int i = 0; i < T; ++i)
      for (int c = 0; c <= i; ++c) {
        const int w = (i + c) % NW;
        ti[w] |= (uint64_t)i << (4 * n[w]);
        tc[w] |= (uint64_t)c << (4 * n[w]);
        rows[w][i >> 2] |= (uint64_t)1 << (16 * (i & 3) + n[w]);
        rows[w][c >> 2] |= (uint64_t)1 << (16 * (c & 3) + n[w]);
        ++n[w];
      }
    most = least = n[0];
    for (int w = 1; w < NW; ++w) {
      most = n[w] > most ? n[w] : most;
      least = n[w] < least ? n[w] : least;
    }
  }
};

template <int T, int W>
struct Elim {
  static constexpr int NW = W == 1 ? 1 : W - 1;   // waves that hold tiles
  static constexpr Deal<T, NW> kDeal{};
  static constexpr int NT = ps::ntiles(T), NS = kDeal.most;
  static_assert(NS <= 16, "tile indices in nibbles");
  int w, lane, c, q, n;
  uint64_t ti, tc, rows0, rows1;   // of the wave, see Deal
  v4d a[NS];

  // tid: the thread's index as of placed_tid
  __device__ __forceinline__ explicit Elim(int tid)
      : w(W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6)), lane(tid & 63), c(tid & 15), q((tid & 63) >> 4),
        n(0), ti(0), tc(0), rows0(0), rows1(0) {
#pragma unroll
    for (int k = 0; k < NW; ++k)
      if (w == k) {
        ti = kDeal.ti[k];
        tc = kDeal.tc[k];
        rows0 = kDeal.rows[k][0];
        rows1 = kDeal.rows[k][1];
        n = kDeal.n[k];
      }
  }
  // 0 .. 63 in the wave for work on vectors, the one that holds no tiles if there
  // is one (its SIMD has no products to wait for), negative in the others
  __device__ __forceinline__ static int vec_tid(int tid) { return tid - 64 * (W - 1); }
  __device__ __forceinline__ bool holds() const { return W == 1 || w < NW; }   // a wave that holds tiles
  __device__ __forceinline__ int tile_i(int s) const { return (int)(ti >> (4 * s)) & 15; }
  __device__ __forceinline__ int tile_c(int s) const { return (int)(tc >> (4 * s)) & 15; }
  __device__ __forceinline__ bool has(int s) const { return s < kDeal.least || s < n; }   // of a wave that holds tiles

  // factor and inverse of the diagonal tile n = -A_JJ; X_JJ to LDS.  The first
  // strip, and the rest
  template <bool LZ>
  __device__ __forceinline__ Diag<LZ> pivot_start(const v4d &n, int J, Lds<T, W> &L, const double *tv) {
    Diag<LZ> g(n, c, q);
    g.template strip<0>(L.scr, L.rs + 16 * J, LZ ? tv + 32 * J : nullptr);
    return g;
  }
  template <bool LZ, class Sink>
  __device__ __forceinline__ v4d pivot_rest(Diag<LZ> &g, int J, Lds<T, W> &L, int *flag, const double *tv, Sink &sink) {
    const double *tz = LZ ? tv + 32 * J : nullptr;
    g.template strip<1>(L.scr, L.rs + 16 * J, tz);
    g.template strip<2>(L.scr, L.rs + 16 * J, tz);
    g.template strip<3>(L.scr, L.rs + 16 * J, tz);
    st_cm(L.xjj(J), c, q, g.e);
    if (LZ && q < 2) L.lzd[32 * J + 2 * c + q] = g.part;
    if constexpr (Sink::kOn) sink.diagonal(J, g.r);
    if (!__all(g.ok) && lane == 0) *flag = 0;
    return g.e;
  }
  template <bool LZ, class Sink>
  __device__ __forceinline__ v4d pivot(const v4d &n, int J, Lds<T, W> &L, int *flag, const double *tv, Sink &sink) {
    Diag<LZ> g = pivot_start<LZ>(n, J, L, tv);
    return pivot_rest<LZ>(g, J, L, flag, tv, sink);
  }

  // The whole elimination of the slots' -A.  Of the pairs bv and tv ([16 T][2],
  // LDS) the first NB are right-hand sides b (consumed) and t = X b; the next
  // NZ of tv are vectors z, and L z is theirs of bv (zero on entry) plus L.lzd.
  // hook(J) runs in step 3 in the waves that hold tiles, when row J of X is
  // complete (X_JC, C < J, at L.row + kTile C, X_JJ at L.xjj(J)).  A sink takes
  // the factor: diagonal(J, L_JJ^T) and below(I, J, rows q + 4 v of L_IJ).  INV
  // false leaves X out (the factor, t and L z only).  flag (LDS) is cleared when
  // a pivot fails.  All 64 W threads call it, after a barrier that follows the
  // caller's writes of bv, tv and flag.
  template <int NB, int NZ, bool INV = true, class Hook, class Sink = NoSink>
  __device__ __forceinline__ void run(Lds<T, W> &L, int *flag, double *bv, double *tv, Hook hook, Sink sink = Sink()) {
    static_assert(NB + NZ <= 2, "one pair of vectors");
    constexpr bool LZ = NZ > 0;
    if constexpr (W == 1) {
      a[0] = pivot<LZ>(a[0], 0, L, flag, tv, sink);
      __syncthreads();
      auto step = [&](int J) __attribute__((always_inline)) {
        if (NB > 0) solve<NB>(J, L, bv, tv);
        row<INV>(J, L, sink);
        __syncthreads();
        hook(J);
        update<INV>(J, L);
        if (NB + NZ > 0) vectors<NB, NZ>(J, L, bv, tv);
        if (J + 1 < T) {
          const int s1 = ps::tix(J + 1, J + 1);
#pragma unroll
          for (int s = 0; s < NS; ++s)
            if (s == s1) a[s] = pivot<LZ>(a[s], J + 1, L, flag, tv, sink);
        }
        __syncthreads();
      };
      if constexpr (T <= 4) {   // the tiles of each step are known
#pragma unroll
        for (int J = 0; J < T; ++J) step(J);
      } else {
#pragma unroll 1
        for (int J = 0; J < T; ++J) step(J);
      }
    } else if (w == NW) {   // the diagonal tiles (the barriers are those of the other branch)
      __syncthreads();
      pivot<LZ>(ld_cm(L.row, c, q), 0, L, flag, tv, sink);
      __syncthreads();
#pragma unroll 1
      for (int J = 0; J < T; ++J) {
        if (NB > 0) solve<NB>(J, L, bv, tv);
        if (J + 1 < T) {
          const v4d xa = neg(ld_rm(L.xjj(J), c, q));
          const v4d r = ln::mfma4(xa, ld_cm(L.dg + kTile, c, q), v4d{0.0, 0.0, 0.0, 0.0});
          Diag<LZ> g = pivot_start<LZ>(ln::mfma4(r, r, ld_cm(L.dg, c, q)), J + 1, L, tv);
          __syncthreads();
          pivot_rest<LZ>(g, J + 1, L, flag, tv, sink);
          if (NB + NZ > 0) vectors<NB, NZ>(J, L, bv, tv);
        } else {
          __syncthreads();
        }
        __syncthreads();
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) a[s] = v4d{0.0, 0.0, 0.0, 0.0};   // (no registers across the loop)
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s)   // what the diagonal tiles 0 and 1 need
        if (has(s) && tile_i(s) <= 1)
          st_cm(tile_i(s) == 0 ? L.row : L.dg + kTile * (1 - tile_c(s)), c, q, a[s]);
      __syncthreads();
      __syncthreads();
#pragma unroll 1
      for (int J = 0; J < T; ++J) {
        // opaque in the loop, so that the addresses formed from the tiles are
        // not kept in registers across it
        asm volatile("" : "+s"(ti), "+s"(tc));
        row<INV>(J, L, sink);
        __syncthreads();
        hook(J);
        update<INV>(J, L);
        __syncthreads();
      }
    }
  }

  // t_J = X_JJ b_J
  template <int NB>
  __device__ __forceinline__ void solve(int J, Lds<T, W> &L, const double *bv, double *tv) const {
    const double t = pair_tdot(ld_pair(bv + 32 * J, c, q), ld_rm(L.xjj(J), c, q));
    if (q < NB) tv[2 * (16 * J + c) + q] = t;
  }

  // 2. row J
  template <bool INV, class Sink>
  __device__ __forceinline__ void row(int J, Lds<T, W> &L, Sink &sink) {
    const double *xj = L.xjj(J);
    const v4d xn = neg(ld_rm(xj, c, q));
    const uint32_t in = (uint32_t)((J < 4 ? rows0 : rows1) >> (16 * (J & 3)));
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (!(in >> s & 1)) continue;
      const int I = tile_i(s), C = tile_c(s);
      if (I == C) {
        if (W > 1 && INV) a[s] = ld_cm(xj, c, q);
      } else if (INV || C == J) {
        const v4d r = ln::mfma4(xn, a[s], v4d{0.0, 0.0, 0.0, 0.0});
        double *o = L.row + kTile * (I + C - J);
        st_cm(o, c, q, r);
        if constexpr (Sink::kOn)
          if (C == J) {
            ln::wave_sync();
            sink.below(I, J, ld_rm(o, c, q));
          }
        a[s] = r;
        if (C == J) a[s] = v4d{0.0, 0.0, 0.0, 0.0};   // Y_IJ starts in step 3
      }
    }
  }

  // b -= R_JI^T t and L z += R_JI^T z for the rows I > J
  template <int NB, int NZ>
  __device__ __forceinline__ void vectors(int J, Lds<T, W> &L, double *bv, const double *tv) const {
    const v4d ty = ld_pair(tv + 32 * J, c, q);
    if constexpr (W == 1) {
#pragma unroll
      for (int I = 1; I < T; ++I) {
        if (I <= J) continue;
        const double e = pair_tdot(ty, ld_cm(L.row + kTile * I, c, q));
        if (q < NB + NZ) {
          double *o = bv + 2 * (16 * I + c) + q;
          *o = q < NB ? *o - e : *o + e;
        }
      }
    } else {   // half of them at a time (those up to row J are multiplied with the others)
      if (J + 1 < T / 2) vectors_of<NB, NZ, 1, T / 2>(J, L, bv, ty);
      vectors_of<NB, NZ, T / 2, T>(J, L, bv, ty);
    }
  }
  template <int NB, int NZ, int I0, int I1>
  __device__ __forceinline__ void vectors_of(int J, Lds<T, W> &L, double *bv, const v4d &ty) const {
    double e[I1 - I0], o[I1 - I0];
#pragma unroll
    for (int I = I0; I < I1; ++I) {
      e[I - I0] = pair_tdot(ty, ld_cm(L.row + kTile * I, c, q));
      o[I - I0] = bv[2 * (16 * I + c) + (q & 1)];
    }
    if (q < NB + NZ) {
#pragma unroll
      for (int I = I0; I < I1; ++I)
        if (I > J) bv[2 * (16 * I + c) + q] = q < NB ? o[I - I0] - e[I - I0] : o[I - I0] + e[I - I0];
    }
  }

  // 3. the tiles below row J, from the last slot (tiles are held row by row: the
  // first one at or above row J ends the loop), the next slot's operands loaded
  // ahead
  template <bool INV>
  __device__ __forceinline__ void update(int J, Lds<T, W> &L) {
    const double *xj = L.xjj(J);
    v4d u, v;
    operands(NS - 1, J, L, xj, u, v);
#pragma unroll
    for (int s = NS - 1; s >= 0; --s) {
      v4d un{}, vn{};
      if (has(s)) {
        const int I = tile_i(s), C = tile_c(s);
        if (I <= J) break;
        if (s > 0) operands(s - 1, J, L, xj, un, vn);
        if (W == 1 || C != J + 1 || I != C) {   // (the next diagonal tile: the fourth wave)
          if (INV || C > J) a[s] = ln::mfma4(u, v, a[s]);
          if (W > 1 && I == J + 2 && C > J) st_cm(L.dg + kTile * (I - C), c, q, a[s]);
        }
      } else {
        operands(s - 1, J, L, xj, un, vn);
      }
      u = un;
      v = vn;
    }
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
    if (!holds()) return;
    constexpr int G = W == 1 ? 1 : 4;   // chains of products at a time
#pragma unroll
    for (int s0 = 0; s0 < NS; s0 += G) {
      v4d yy[G];
      double u[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        u[g] = 0.0;
        if (s0 + g < NS) yy[g] = ld_pair(y + 32 * tile_i(s0 + g), c, q);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (s0 + g < NS) u[g] = __builtin_amdgcn_mfma_f64_4x4x4f64(yy[g][k], a[s0 + g][k], u[g], 0, 0, 0);
      if (q < 2) {
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (s0 + g < NS && has(s0 + g))
            part[ps::tix(tile_i(s0 + g), tile_c(s0 + g)) * 32 + 16 * q + c] = u[g];
      }
    }
  }
  // the squared columns of X likewise, to part[tix(I, C)][16]
  __device__ __forceinline__ void xsq(double *part) const {
    if (!holds()) return;
    const v4d one{1.0, 1.0, 1.0, 1.0};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (!has(s)) continue;
      const double u = pair_tdot(one, a[s] * a[s]);
      if (q == 0) part[ps::tix(tile_i(s), tile_c(s)) * 16 + c] = u;
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
  if (!E.holds()) return;
#pragma unroll
  for (int s = 0; s < Elim<T, W>::NS; ++s) {
    if (!E.has(s)) continue;
    const int I = E.tile_i(s), C = E.tile_c(s);
    double *o = xo + (cix<T>(C) + 16 * (I - C)) * 16;   // (the same in all lanes)
#pragma unroll
    for (int v = 0; v < 4; ++v) o[(unsigned)E.lane + 64 * v] = E.a[s][v];
  }
}

}  // namespace el
