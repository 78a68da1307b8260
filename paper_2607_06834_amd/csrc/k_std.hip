// Kernels of the standardized form (Sec. IV.B; Eqs. PTA_standard_transform_curn,
// standardized_stochastic_posterior in the Gram form of Eq. posterior_implemented;
// App. B for a tempered likelihood).
//
// Per pulsar I and chain c (one workgroup each):
//   A = beta S0_I + diag(1 / D),  D = CURN variances of the chain (rho_k + kappa_Ik,
//   kappa_dm,Ik);  Sigma = A^-1 = L L^T with L the lower Cholesky factor.
// In the reversed index order r = P - 1 - j the matrix A~ = J A J has a lower
// Cholesky factor L~, and L = J L~^-T J: the lower Cholesky factor of the
// covariance comes from the ordinary factorisation of the reversed precision.
// With X = L~^-1 (lower):
//   a~ = X^T (X beta d~ + z~)      (a = a_hat + L z)
//   ln det L = sum_r ln X_rr
// The adjoint (k_std_bwd) takes v = dF/da = beta (d - S0 a) - phi^-1 a:
//   dlogp/dz~ = X v~
//   dlogp/dD_j = [a_hat_j (Sigma v)_j + T_j + Sigma_jj / 2] / D_j^2
// with (Sigma v)~ = X^T X v~, Sigma~_rr = |X e_r|^2 and T_r a suffix sum down
// column r of X (the diagonal of L Phi(L^T v z^T) L^T).
//
// Per frequency k and chain (k_std_prior): phi_k = rho_k Gamma + diag kappa_.k
// (Eq. prior_cov) factorised the same way, y = X_k a, u = X_k^T y = phi_k^-1 a,
// and the explicit prior derivatives 1/2 u^T Gamma u - tr(phi_k^-1 Gamma) (rho)
// and 1/2 u_I^2 - (phi_k^-1)_II (kappa), with tr(phi^-1 Gamma) = |X_k chol Gamma|_F^2.
//
// With a deterministic CW in its own basis (Sec. IV.C), k_std_cw_fwd replaces
// d and dt^T N~^-1 dt of each (pulsar, chain) by those of dt - F_D a_D before
// the transform, and k_std_cw_bwd takes dlog p / d d_bar = beta (a + Sigma v)
// (the likelihood's explicit term plus the shift of a_hat) back to the CW
// parameters through S_D, Q_D, e_D, the transform of the samples and the
// waveform's derivative.
//
// X = L~^-1 is formed by block Gauss-Jordan elimination with the matrix in the
// registers of one to three waves (elim_dev.h), which carries t = X beta d~ and
// L~ z~ along.  What bounds it: at 67 pulsars x 64 chains (T = 8) the products of
// a problem take 57e3 cycles of a matrix core, a third of that on each of three
// SIMDs; k_std_fwd<8> runs at half of the matrix cores' cycles there, held by what
// elim_dev.h says, and X goes to memory (309 MB, 68 us).  The earlier form, with
// the tiles in LDS (two problems a compute unit, every operand and result through
// LDS), took 525 us a launch where this takes 253, 335 where this takes 84 at 100
// pulsars with T = 4, and k_split_fac<8> 466 where this takes 236.
#include <cmath>

#include "cw_dev.h"
#include "elim_dev.h"
#include "std.h"

namespace {

using ps::StdDev;
using ln::v4d;

// Waves per (pulsar, chain) or (frequency, chain) elimination of T tiles, and the
// waves a SIMD that its registers are held to.  One wave takes at most 15 tiles
// (120 of its registers); from T = 6 three waves share them and a fourth takes the
// diagonal tiles.  Measured, us: T = 7 for 900, at three waves a SIMD
// 102, at four (six registers spilled outside of the steps) 88; T = 8 for 4288, at
// three 254, at four 296 (142 registers spilled).
// The prior's problems are fewer and do more at each step: T = 5 with one wave and
// with four for 112 problems 39 and 23, for 896 63 and 50, for 3584 145 and 143;
// T = 4 28 and 38 for 896 (and k_std_fwd<5>, 4288 problems, 78 and 96).
template <int T>
constexpr int elim_waves() { return T <= 5 ? 1 : 4; }
template <int T>
constexpr int prior_waves() { return T <= 4 ? 1 : 4; }
template <int T>
constexpr int prior_occ() { return T == 4 ? 2 : T == 3 || T == 8 ? 3 : 4; }
template <int T>
constexpr int elim_occ() { return T <= 2 || T == 6 || T == 7 ? 4 : T == 5 ? 2 : 3; }

// the plain row-major tile t of global memory as an MFMA B operand
__device__ inline v4d ldg_cm(const double *t, int c, int q) {
  const double *p = t + 16 * q + c;
  return v4d{p[0], p[64], p[128], p[192]};
}

// Block sum of one value per thread (W waves); every thread gets the sum.  tid is
// the index by which the threads share the work (placed_tid): the waves' parts
// are added in its order, whichever SIMDs they run on.
template <int W>
__device__ inline double wave_block_sum(double v, double *red, int tid) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if (W == 1) return v;
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double s = red[0];
#pragma unroll
  for (int i = 1; i < W; ++i) s += red[i];
  return s;
}

// Block sum of one value per thread (256 threads); every thread gets the sum.
__device__ inline double block_sum(double v, double *red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int tid = threadIdx.x;
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Problem index of block b in a grid of n: consecutive blocks are dealt to
// the 8 XCDs in turn, so XCD x = b % 8 is given the x-th contiguous range of
// problem indices (with pulsar-major problems, a few pulsars' data per L2).
__device__ inline int xcd_index(int b, int n) {
  const int x = b & 7, k = b >> 3, q = n >> 3, rm = n & 7;
  return x * q + (x < rm ? x : rm) + k;
}

// sum over a wave
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The slots of a wave that holds tiles from S0~ (rows of block C, columns of
// block I, every load issued before any use), and -(beta S0~ + diag(1 / D~)) of
// them.  In a wave that waits for another's matrix instructions an FP64 operation
// costs up to 64 cycles: the sign is changed without one, and beta = 1 takes none.
template <int T, class E>
__device__ __forceinline__ void load_gram(E &el, const double *__restrict__ s0) {
  constexpr int pp = 16 * T;
  if (!el.holds()) return;
  const unsigned l = el.q * pp + el.c;
#pragma unroll
  for (int s = 0; s < E::NS; ++s) {
    const double *t = s0 + (el.has(s) ? 16 * (el.tile_c(s) * pp + el.tile_i(s)) : 0);   // (the same in all lanes)
#pragma unroll
    for (int v = 0; v < 4; ++v) el.a[s][v] = t[l + 4 * v * pp];
  }
}
template <int T, class E>
__device__ __forceinline__ void gram_slots(E &el, double beta, const double *di) {
  if (!el.holds()) return;
  if (beta != 1.0) {
#pragma unroll
    for (int s = 0; s < E::NS; ++s) el.a[s] *= beta;
  }
#pragma unroll
  for (int s = 0; s < E::NS; ++s) {
    el.a[s] = el::neg(el.a[s]);
    if (el.tile_i(s) == el.tile_c(s)) {
      const double d = di[16 * el.tile_i(s) + el.c];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (el.q + 4 * v == el.c) el.a[s][v] -= d;
    }
  }
}

// ---------------------------------------------------------------------------
// Forward per (pulsar, chain): transform, likelihood, Jacobian.
// ---------------------------------------------------------------------------
template <int T>
__global__ __launch_bounds__(64 * elim_waves<T>(), elim_occ<T>()) void k_std_fwd(StdDev S, const double *__restrict__ x) {
  constexpr int W = elim_waves<T>(), pp = 16 * T;
  using E = el::Elim<T, W>;
  __shared__ el::Lds<T, W> L;
  __shared__ double bv[2 * pp], tv[2 * pp], vdi[pp], dv[W > 1 ? pp : 1];   // (b, L z), (t, z), 1 / D~, d
  __shared__ int flag;
  const int tid = el::placed_tid<W>();
  const int pi = xcd_index(blockIdx.x, gridDim.x);
  const int I = pi / S.n_chains, c = pi - I * S.n_chains;
  const double *xc = x + (size_t)c * S.d;
  const double beta = S.beta ? S.beta[c] : 1.0;
  const int P = S.P;
  const size_t ci = (size_t)c * S.n_psr + I;
  E el(tid);
  // A~ = beta S0~ + diag(1 / D~)
  load_gram<T>(el, S.s0 + (size_t)I * pp * pp);
  // d of the data, or of the data minus the deterministic signal; vectors in the
  // wave that holds no tiles
  const double *dsrc = S.has_cw ? S.dbar + ci * pp : S.dvec + (size_t)I * pp;
  const int vt = E::vec_tid(tid);
  if (vt >= 0) {
    bool bad = false;
#pragma unroll
    for (int u = 0; u < (pp + 63) / 64; ++u) {
      const int r = vt + 64 * u;
      if (r >= pp) break;
      const double d = (r < P) ? dsrc[r] : 0.0;
      if (W > 1) dv[r] = d;
      bv[2 * r] = beta * d;
      bv[2 * r + 1] = 0.0;
      // with split coefficients this is the combined MAP only (z = 0)
      tv[2 * r + 1] = (r < P && !S.split) ? xc[S.off_z + I * P + (P - 1 - r)] : 0.0;
      if (r >= P) vdi[r] = 1.0;
    }
    // a CURN variance that is not positive and finite leaves phi_CURN not positive
    // definite; a lane per frequency, for the sine and the cosine row
    static_assert(pp <= 128, "a lane per frequency");
    if (2 * vt < P) {
      const double Dv = ps::curn_var(S, xc, I, 2 * vt);
      bad = !(Dv > 0.0 && isfinite(Dv));
      const double di = 1.0 / Dv;
      vdi[P - 1 - 2 * vt] = di;
      vdi[P - 2 - 2 * vt] = di;
    }
    bad = __any(bad);
    if (vt == 0) flag = bad ? 0 : 1;
  }
  __syncthreads();
  gram_slots<T>(el, beta, vdi);
  __syncthreads();
  // X = L~^-1, t = X beta d~ and L~ z~
  el.template run<1, 1>(L, &flag, bv, tv, [](int) {});
  if (vt >= 0)
    for (int r = vt; r < pp; r += 64) tv[2 * r + 1] += tv[2 * r];
  __syncthreads();
  // a_hat~ = X^T t, a~ = X^T (t + z~)
  double *part = L.row;
  static_assert(E::NT * 32 <= T * el::kTile, "the partial sums fit the row buffer");
  el.xty(part, tv);
  __syncthreads();
  el::store_x(el, S.xinv + ci * (E::NT * 256));
  if (vt < 0) return;
  double part_d = 0.0, part_v = 0.0, part_j = 0.0;
  for (int r = vt; r < pp; r += 64) {
    const double sh = el::xty_sum<T, 2>(part, 0, r), sa = el::xty_sum<T, 2>(part, 1, r);
    S.ahat[ci * pp + r] = sh;
    // beta (d - S0 a) in the reversed order: A~ a~ = L~ (t + z~) = beta d~ + L~ z~,
    // so beta S0~ a~ = beta d~ + L~ z~ - a~ / D~ and v1 = a~ / D~ - L~ z~
    const double v1 = sa * vdi[r] - (bv[2 * r + 1] + L.lzd[2 * r + 1]);
    S.v1[ci * pp + r] = v1;
    if (r < P) {
      S.avec[ci * pp + (P - 1 - r)] = sa;
      part_d += sa * (W > 1 ? dv[r] : dsrc[r]);
      part_j += log(L.rs[r]);
    }
    part_v += sa * v1;
  }
  part_d = wave_sum(part_d);
  part_v = wave_sum(part_v);
  part_j = wave_sum(part_j);
  if (vt == 0) {
    // beta log L = beta (-dt N~^-1 dt / 2 + a.d - a.S0 a / 2 + c1), with
    // beta a.S0 a = beta a.d - a.v1
    const double *k2 = S.cconst + 2 * I;
    const double c0 = S.has_cw ? S.cbar[ci] : k2[0];
    double *o = S.lik + ci * 2;
    o[0] = beta * (k2[1] - 0.5 * c0) + 0.5 * beta * part_d + 0.5 * part_v;
    o[1] = part_j;
    S.flag1[ci] = flag ? 0 : ps::kFlagNotPD;
  }
}

// ---------------------------------------------------------------------------
// Prior of the diagonal items: red-noise frequencies beyond the common process
// (phi_k = diag kappa_.k) and DM (diag kappa_dm): one thread per (chain, pulsar,
// item), items k in [nf_gw, ka) then the DM frequencies.  With split
// coefficients: the whole pulsar-noise set a_R, items k < nf_rn then DM.  With a
// common process they are workgroups after its problems in the same launch (the
// two write different entries, and they run on what the problems leave free).  In
// a launch of their own they took 5 to 8 us, a tenth of an evaluation of 20 pulsars
// x 8 chains (ten leapfrogs 461 us, so 436); the dense launch is 1 us longer for
// them at 67 pulsars x 64 chains, k_split_prior_g 2.5.
// ---------------------------------------------------------------------------
__device__ inline size_t prior_diag_items(const StdDev &S) {
  return (size_t)S.n_chains * S.n_psr * ((S.split ? S.nf_rn : S.ka - S.nf_gw) + S.kdm);
}
__device__ __forceinline__ void prior_diag_item(const StdDev S, const double *__restrict__ x, size_t e) {
  const int k0 = S.split ? 0 : S.nf_gw;
  const int nrn = S.split ? S.nf_rn : S.ka - S.nf_gw, per = nrn + S.kdm;
  const int it = (int)(e % per);
  const size_t ci = e / per;
  const int I = (int)(ci % S.n_psr), c = (int)(ci / S.n_psr);
  const double *xc = x + (size_t)c * S.d;
  int k, col;
  double kap;
  if (it < nrn) {
    k = k0 + it;
    col = 2 * k;
    kap = ps::spec_value(S, xc, 1, I, k);
  } else {
    k = it - nrn;
    col = (S.split ? 2 * S.nf_rn : 2 * S.ka) + 2 * k;   // row in a_R, or in a
    kap = ps::spec_value(S, xc, 2, I, k);
  }
  const double *av = S.split ? S.ar + ci * S.ppr : S.avec + ci * S.pp;
  const double a0 = av[col], a1 = av[col + 1];
  const double ik = 1.0 / kap;
  const double u0 = a0 * ik, u1 = a1 * ik;
  double *v2 = S.split ? S.v2r + ci * S.ppr : S.v2 + ci * S.pp;
  v2[col] = -u0;
  v2[col + 1] = -u1;
  const double dk = 0.5 * (u0 * u0 + u1 * u1) - ik;
  if (it < nrn) S.dkap_e[((size_t)c * S.n_psr + I) * S.ka + k] = dk;
  else S.ddm_e[((size_t)c * S.n_psr + I) * S.kdm + k] = dk;
  double *o = S.diag_q + (((size_t)c * S.n_psr + I) * (S.ka + S.kdm) + (it < nrn ? k : S.ka + k)) * 2;
  o[0] = a0 * u0 + a1 * u1;
  o[1] = log(kap);
  S.flag3[((size_t)c * S.n_psr + I) * (S.ka + S.kdm) + (it < nrn ? k : S.ka + k)] =
      ((kap > 0.0) && isfinite(kap)) ? 0 : ps::kFlagNotPD;
}

__global__ __launch_bounds__(256) void k_std_prior_diag(StdDev S, const double *__restrict__ x) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e < prior_diag_items(S)) prior_diag_item(S, x, e);
}

// the workgroups of NTH threads after the n_dense ones of a launch
template <int NTH>
__device__ __forceinline__ bool prior_diag_group(const StdDev &S, const double *__restrict__ x, int n_dense) {
  if ((int)blockIdx.x < n_dense) return false;
  const size_t e = (size_t)(blockIdx.x - n_dense) * NTH + threadIdx.x;
  if (e < prior_diag_items(S)) prior_diag_item(S, x, e);
  return true;
}

// ---------------------------------------------------------------------------
// Prior per (frequency k < nf_gw, chain): phi_k = rho_k Gamma + diag kappa_.k.
// ---------------------------------------------------------------------------
template <int T>
__global__ __launch_bounds__(64 * prior_waves<T>(), prior_occ<T>()) void k_std_prior_dense(StdDev S,
                                                                                    const double *__restrict__ x) {
  constexpr int W = prior_waves<T>(), pp = 16 * T, NTH = 64 * W;
  if (prior_diag_group<NTH>(S, x, S.n_chains * S.nf_gw)) return;
  using E = el::Elim<T, W>;
  __shared__ el::Lds<T, W> L;
  __shared__ double bv[2 * pp], tv[2 * pp], vk[pp], red[W], rho_l;   // a then u, y = X a (sin, cos)
  __shared__ int flag;
  const int tid = el::placed_tid<W>();
  const int c = blockIdx.x / S.nf_gw, k = blockIdx.x - c * S.nf_gw;
  const int n = S.n_psr;
  const double *xc = x + (size_t)c * S.d;
  E el(tid);
#pragma unroll
  for (int s = 0; s < E::NS; ++s) {
    // Gamma is stored as lower tiles: the slot takes rows of block C, columns
    // of block I, the transposed tile
    const double *g = S.gam_tiles + (el.has(s) ? ps::tix(el.tile_i(s), el.tile_c(s)) : 0) * 256 + 16 * el.c + el.q;
#pragma unroll
    for (int v = 0; v < 4; ++v) el.a[s][v] = g[4 * v];
  }
  const int vt = E::vec_tid(tid);
  if (vt >= 0) {
    const double r = ps::spec_value(S, xc, 0, 0, k);
#pragma unroll
    for (int u = 0; u < (pp + 63) / 64; ++u) {
      const int i = vt + 64 * u;
      if (i >= pp) break;
      const double *av = S.avec + ((size_t)c * n + i) * S.pp;
      vk[i] = (i < n) ? ((k < S.nf_rn) ? ps::spec_value(S, xc, 1, i, k) : 0.0) : 1.0;
      bv[2 * i] = (i < n) ? av[2 * k] : 0.0;
      bv[2 * i + 1] = (i < n) ? av[2 * k + 1] : 0.0;
    }
    if (vt == 0) {
      flag = 1;
      rho_l = r;
    }
  }
  __syncthreads();
  const double rho = rho_l;
#pragma unroll
  for (int s = 0; s < E::NS; ++s) {
    const bool dg = el.tile_i(s) == el.tile_c(s);
    const double kv = dg ? vk[16 * el.tile_i(s) + el.c] : 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      el.a[s][v] = -fma(rho, el.a[s][v], (dg && el.q + 4 * v == el.c) ? kv : 0.0);
  }
  // X and y = X a for sin and cos; tr(phi^-1 Gamma) = |X G|_F^2, G = chol(Gamma),
  // row by row as X is formed: tiles (X G)_JK = sum_{M=K}^{J} X_JM G_MK
  double part_t = 0.0;
  el.template run<2, 0>(L, &flag, bv, tv, [&](int J) {
    for (int K = (el.w + J) % E::NW; K <= J; K += E::NW) {
      v4d r{0.0, 0.0, 0.0, 0.0};
      for (int M = K; M <= J; ++M) {
        const v4d g = ldg_cm(S.gch_tiles + ps::tix(M, K) * 256, el.c, el.q);
        r = ln::mfma4(el::ld_rm(M < J ? L.row + el::kTile * M : L.xjj(J), el.c, el.q), g, r);
      }
      part_t += (r[0] * r[0] + r[1] * r[1]) + (r[2] * r[2] + r[3] * r[3]);
    }
  });
  // u = X^T y and the squared columns of X
  double *part = L.row;
  static_assert(E::NT * 48 <= T * el::kTile, "the partial sums fit the row buffer");
  el.xty(part, tv);
  el.xsq(part + E::NT * 32);
  __syncthreads();
  double part_q = 0.0, part_l = 0.0;
  for (int i = tid; i < pp; i += NTH) {
    bv[2 * i] = el::xty_sum<T, 2>(part, 0, i);
    bv[2 * i + 1] = el::xty_sum<T, 2>(part, 1, i);
    vk[i] = el::xty_sum<T, 1>(part + E::NT * 32, 0, i);   // (phi^-1)_II
    part_q += tv[2 * i] * tv[2 * i] + tv[2 * i + 1] * tv[2 * i + 1];
    if (i < n) part_l -= 2.0 * log(L.rs[i]);
  }
  __syncthreads();
  // Gamma u (columns of the symmetric Gamma, coalesced) for the rho term,
  // eight loads in flight at a time
  double part_g = 0.0;
  for (int e = tid; e < 2 * pp; e += NTH) {
    const int i = e % pp, h = e / pp;
    if (i < n) {
      double s = 0.0;
      int m = 0;
      for (; m + 8 <= n; m += 8) {
        double g[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) g[u] = S.gamma[(size_t)(m + u) * n + i];
#pragma unroll
        for (int u = 0; u < 8; ++u) s = fma(g[u], bv[2 * (m + u) + h], s);
      }
      for (; m < n; ++m) s = fma(S.gamma[(size_t)m * n + i], bv[2 * m + h], s);
      part_g += s * bv[2 * i + h];
    }
  }
  const double quad = wave_block_sum<W>(part_q, red, tid);
  const double ldet = wave_block_sum<W>(part_l, red, tid);
  const double ugu = wave_block_sum<W>(part_g, red, tid);
  const double tr = wave_block_sum<W>(part_t, red, tid);
  for (int i = tid; i < n; i += NTH) {
    const double u0 = bv[2 * i], u1 = bv[2 * i + 1];
    S.dkap_e[((size_t)c * n + i) * S.ka + k] = 0.5 * (u0 * u0 + u1 * u1) - vk[i];
    double *v2 = S.v2 + ((size_t)c * n + i) * S.pp;
    v2[2 * k] = -u0;
    v2[2 * k + 1] = -u1;
  }
  if (tid == 0) {
    double *o = S.quad_k + ((size_t)c * S.ka + k) * 2;
    o[0] = quad;
    o[1] = ldet;
    S.drho_e[(size_t)c * S.ka + k] = 0.5 * ugu - tr;
    S.flag2[(size_t)c * S.ka + k] = flag ? 0 : ps::kFlagNotPD;
  }
}

// ---------------------------------------------------------------------------
// Adjoint per (pulsar, chain): dlogp/dz and dlogp/dD.
// ---------------------------------------------------------------------------

// Lane l ^ (2 M - 1) of a 16-lane row, M = 8, 4, 2, 1: the mirror of the row,
// of its halves, of its quads, of its pairs (DPP).
template <int M>
__device__ inline double mirror_d(double v) {
  constexpr int ctrl = M == 8 ? 0x140 : M == 4 ? 0x141 : M == 2 ? 0x1B : 0xB1;
  const long long b = __double_as_longlong(v);
  return ln::join_d(__builtin_amdgcn_update_dpp(0, (int)b, ctrl, 0xF, 0xF, false),
                    __builtin_amdgcn_update_dpp(0, (int)(b >> 32), ctrl, 0xF, 0xF, false));
}

// Sums of N = 16, 8 or 4 values over the 16 lanes of a row: lane c ends with
// the sum of value c N / 16 (halves of the values go to the two halves of the
// lanes until one is left).
template <int N>
__device__ __forceinline__ double row_sums(double (&v)[N], int c) {
  if (N >= 2) {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const bool up = c & 8;
      v[i] = (up ? v[i + N / 2] : v[i]) + mirror_d<8>(up ? v[i] : v[i + N / 2]);
    }
  }
#pragma unroll
  for (int i = 0; i < N / 4; ++i) {
    const bool up = c & 4;
    v[i] = (up ? v[i + N / 4] : v[i]) + mirror_d<4>(up ? v[i] : v[i + N / 4]);
  }
  if (N >= 8) {
#pragma unroll
    for (int i = 0; i < N / 8; ++i) {
      const bool up = c & 2;
      v[i] = (up ? v[i + N / 8] : v[i]) + mirror_d<2>(up ? v[i] : v[i + N / 8]);
    }
  } else {
    v[0] += mirror_d<2>(v[0]);
  }
  if (N >= 16) {
    const bool up = c & 1;
    v[0] = (up ? v[1] : v[0]) + mirror_d<1>(up ? v[0] : v[1]);
  } else {
    v[0] += mirror_d<1>(v[0]);
  }
  return v[0];
}

// The sums of a column over its rows a, top to bottom, that the adjoint needs:
// sv = sum X_ar w_a, ss = sum X_ar^2, suf = sum X_ar z_a and
// tt = sum_a X_ar w_a (sum_{b>a} X_br z_b + X_ar z_a / 2).
struct ColSum {
  double sv, ss, suf, tt;
  __device__ inline void below(const ColSum &o) {   // this column's rows, then those of o
    tt += o.tt + sv * o.suf;
    sv += o.sv;
    ss += o.ss;
    suf += o.suf;
  }
};

// The adjoint reads all of X once (316 MB a launch at 67 pulsars x 64 chains,
// T = 8), which bounds it.  It takes the problems in the reverse of the order in
// which the forward wrote them, so that the 256 MB memory-side cache still holds
// most of what it reads: 67 us there (4.7 TB/s), in the forward's order 95
// (3.3 TB/s); through LDS, two problems a compute unit and a thread per half row
// and half column, 136.  k_split_bwd likewise 73 and 106; k_split_bwd_c, whose X
// is older than another set's, finds little of it in either order (98 us; 88 with
// k_split_bwd in the forward's order).
//
// X of one problem (block columns of 16, see el::store_x) in registers: wave w
// of (T + 1) / 2 takes the block columns w and T - 1 - w, 4 (T + 1) values a lane
// in all (half of that for the middle one of an odd T), so that the waves are
// even.  Lane (c, q) holds a quarter q of the rows of column c, consecutive
// ones: the sums down a column run in one lane and only their four parts are
// put together across lanes.  X is read once, 128 bytes a row of 16 lanes.
template <int T>
struct AdjX {
  static constexpr int W = (T + 1) / 2, NI = 4 * (T + 1), pp = 16 * T;
  int w, c, q, C2, n1, n2;
  double x[NI];

  __device__ __forceinline__ AdjX(const double *__restrict__ xi, int tid)
      : w(W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6)), c(tid & 15), q((tid & 63) >> 4), C2(T - 1 - w),
        n1(4 * (T - w)), n2(C2 != w ? 4 * (w + 1) : 0) {
    const double *p1 = xi + (el::cix<T>(w) + q * n1) * 16 + c;
    const double *p2 = xi + (el::cix<T>(C2) + q * n2 - n1) * 16 + c;
#pragma unroll
    for (int k = 0; k < NI; ++k) x[k] = k < n1 ? p1[k * 16] : k < n1 + n2 ? p2[k * 16] : 0.0;
  }
  __device__ inline int row_of(int k) const { return k < n1 ? 16 * w + q * n1 + k : 16 * C2 + q * n2 + k - n1; }

  // This wave's part of X v by rows to wp[T][pp] (LDS): row r over block column
  // C in wp[C][r]; after a barrier row_total adds a row's block columns in order.
  template <int N>
  __device__ __forceinline__ void rows_part(int k0, const double v1, const double v2, double *wp) {
    double p[N];
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = x[k0 + i] * (k0 + i < n1 ? v1 : v2);
    const double s = row_sums<N>(p, c);
    const int k = k0 + c * N / 16;
    if (c % (16 / N) == 0 && k < n1 + n2) wp[(k < n1 ? w : C2) * pp + row_of(k)] = s;
  }
  __device__ __forceinline__ void rows(const double *v, double *wp) {
    const double v1 = v[16 * w + c], v2 = v[16 * C2 + c];
    constexpr int n16 = NI / 16;
#pragma unroll
    for (int g = 0; g < n16; ++g) rows_part<16>(16 * g, v1, v2, wp);
    if constexpr (NI % 16 >= 8) rows_part<8>(16 * n16, v1, v2, wp);
    if constexpr (NI % 8 >= 4) rows_part<4>(NI - 4, v1, v2, wp);
  }
  static __device__ inline double row_total(const double *wp, int r) {
    double s = 0.0;
    for (int C = 0; C <= (r >> 4); ++C) s += wp[C * pp + r];
    return s;
  }

  // Column sums of the wave's block columns: sink(column, sums) in the lanes
  // of row 0, wz[r] = (w_r, z_r) (LDS).
  template <class Sink>
  __device__ __forceinline__ void columns(const double2 *wz, Sink sink) {
    ColSum s{0.0, 0.0, 0.0, 0.0}, s2{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = NI - 1; k >= 0; --k) {
      if (k >= n1 + n2) continue;
      if (k == n1 - 1) {   // the second block column is done
        s2 = s;
        s = ColSum{0.0, 0.0, 0.0, 0.0};
      }
      const double2 a = wz[row_of(k)];
      const double xv = x[k], xw = xv * a.x;
      s.tt = fma(xw, fma(0.5 * xv, a.y, s.suf), s.tt);
      s.sv += xw;
      s.ss = fma(xv, xv, s.ss);
      s.suf = fma(xv, a.y, s.suf);
    }
    finish(s, w, sink);
    if (n2 > 0) finish(s2, C2, sink);
  }
  template <class Sink>
  __device__ __forceinline__ void finish(ColSum s, int C, Sink sink) {
    // quarters q, q ^ 1 and then the halves, the upper rows first
#pragma unroll
    for (int m = 1; m <= 2; m *= 2) {
      const bool lower = q & m;
      const ColSum o = m == 1 ? ColSum{ln::xor16_d(s.sv, q), ln::xor16_d(s.ss, q), ln::xor16_d(s.suf, q),
                                       ln::xor16_d(s.tt, q)}
                              : ColSum{ln::xor32_d(s.sv, q), ln::xor32_d(s.ss, q), ln::xor32_d(s.suf, q),
                                       ln::xor32_d(s.tt, q)};
      ColSum u = lower ? o : s;
      u.below(lower ? s : o);
      s = u;
    }
    if (q == 0) sink(16 * C + c, s);
  }
};

template <int T>
__global__ __launch_bounds__(64 * AdjX<T>::W, 4) void k_std_bwd(StdDev S, const double *__restrict__ x,
                                                             double *__restrict__ grad) {
  constexpr int W = AdjX<T>::W, pp = 16 * T, NTH = 64 * W;
  __shared__ double wp[T * pp], vv[pp], gd[pp], sg[pp];
  __shared__ double2 wz[pp];
  const int tid = threadIdx.x;
  const int pi = (int)gridDim.x - 1 - xcd_index(blockIdx.x, gridDim.x);   // the latest X first
  const int I = pi / S.n_chains, c = pi - I * S.n_chains;
  const double *xc = x + (size_t)c * S.d;
  const int P = S.P;
  const size_t ci = (size_t)c * S.n_psr + I, vb = ci * pp;
  AdjX<T> X(S.xinv + ci * (ps::ntiles(T) * 256), tid);
  static_assert(NTH >= pp, "a thread per row");
  const int r = tid;
  double zr = 0.0, ah = 0.0, Dv = 1.0;
  if (r < pp) {
    vv[r] = (r < P) ? S.v1[vb + r] + S.v2[vb + (P - 1 - r)] : 0.0;
    if (r < P) {
      zr = xc[S.off_z + I * P + (P - 1 - r)];
      ah = S.ahat[vb + r];
      Dv = ps::curn_var(S, xc, I, P - 1 - r);
    }
  }
  __syncthreads();
  // w~ = X v~ (dlogp/dz~)
  X.rows(vv, wp);
  __syncthreads();
  if (r < pp) {
    const double s = AdjX<T>::row_total(wp, r);
    wz[r] = double2{s, zr};
    if (r < P) grad[(size_t)c * S.d + S.off_z + I * P + (P - 1 - r)] = s;
  }
  __syncthreads();
  // per column r: (Sigma v)~_r, Sigma~_rr and T_r;
  // dlogp/dD~_r = (a_hat~_r (Sigma v)~_r + T_r + Sigma~_rr / 2) / D~_r^2
  X.columns(wz, [&](int col, const ColSum &s) {
    sg[col] = s.sv;
    gd[col] = s.tt + 0.5 * s.ss;
  });
  __syncthreads();
  if (r < P) {
    gd[r] = fma(ah, sg[r], gd[r]) / (Dv * Dv);
    if (S.has_cw) {
      // dlog p / d d_bar (original order): beta a (likelihood) + beta Sigma v (a_hat)
      const double beta = S.beta ? S.beta[c] : 1.0;
      const int j = P - 1 - r;
      S.gdbar[ci * P + j] = beta * (S.avec[vb + j] + sg[r]);
    }
  }
  __syncthreads();
  if (tid < S.ka + S.kdm) {
    const int r0 = P - 1 - 2 * tid, r1 = r0 - 1;   // the DM block follows the red/common one
    const double g = gd[r0] + gd[r1];
    if (tid < S.ka) S.dD_rn[ci * S.ka + tid] = g;
    else S.dD_dm[ci * S.kdm + (tid - S.ka)] = g;
  }
}

// ---------------------------------------------------------------------------
// Deterministic CW in its own basis (Sec. IV.C), per (pulsar, chain).
// ---------------------------------------------------------------------------
__device__ inline pt::CwLane cw_lane(const double cst[pt::kCwRows]) {
  pt::CwLane L;
  L.K1 = cst[pt::kCwK1];
  L.inv32X = cst[pt::kCwInv32X];
  L.phi0 = cst[pt::kCwPhi0];
  L.a0 = cst[pt::kCwA0];
  L.ci = cst[pt::kCwCi];
  L.U = cst[pt::kCwU];
  L.V = cst[pt::kCwV];
  L.c2s = cst[pt::kCwC2s];
  L.s2s = cst[pt::kCwS2s];
  return L;
}

// The CW kernels take a pulsar and a block of kCwChains = 16 chains per workgroup
// of eight waves: each table (the transform, S_D, Q_D) is one operand of matrix
// products with the chains as the other's 16 columns, a wave per 16 rows.
// Vectors of the block lie in LDS as [row][16 chains], rows of kCwLd doubles
// (lanes 16 apart read rows four apart: other halves of the banks), zero beyond
// their length.  What bounds them: the 96 matrix instructions a wave, two
// workgroups on more than half of the compute units at 100 pulsars x 64 chains
// (11 us), and the waveform ahead of them; the tables are loaded a product ahead.
// With a table row per thread and vector FMAs (eight LDS reads a table entry)
// they took 53 and 50 us there, with four waves and the tables loaded where
// they are used 32 and 35, now 27 and 29.
constexpr int kCwChains = 16, kCwLd = 20, kCwRowsMax = 16 * ((ps::kMaxCwM + 15) / 16), kCwT = 512;

// Constants of the block's chains for pulsar I (cst: kCwChains x kCwRows, LDS):
// wave 0 the orbit, its three powers of ten in groups of 16 lanes, wave 1 the sky
// position, its two sines likewise (a chain's constants in one lane are a serial
// chain of about 4 us).
__device__ inline void cw_block_constants(const StdDev &S, const double *x, int I, int c0, int nc,
                                          double *cst) {
  const int tid = threadIdx.x, l = tid & 63, ch = l & 15, g = l >> 4;
  if (tid >= 128) return;
  const double *th = x + (size_t)(c0 + min(ch, nc - 1)) * S.d + S.off_cw;
  double *o = cst + ch * pt::kCwRows;
  if (tid < 64) {
    const double e = exp(pt::kLn10 * th[g == 0 ? 2 : g == 1 ? 3 : 7]);
    const double f10 = __shfl(e, 16 + ch, 64), h10 = __shfl(e, 32 + ch, 64);
    if (g == 0) pt::cw_orbit(th, e, f10, h10, o);
  } else {
    double sn, cs;
    sincos(g == 0 ? 2.0 * th[6] : th[1], &sn, &cs);
    const double sph = __shfl(sn, 16 + ch, 64), cph = __shfl(cs, 16 + ch, 64);
    if (g == 0) pt::cw_sky(th[0], S.cw_pos + 3 * I, sn, cs, sph, cph, o);
  }
}

// Four 16-column blocks of 16 rows of a table as operands of sixteen products:
// lane (c, q) holds row r0 + c, columns 16 (b + u) + 4 q + i in a[4 u + i], so
// that a row-major table (ks = 1) is read in runs of four.  Element (row, k) is
// at row rs + k ks; rows past nr and columns past nk repeat the last, blocks
// past nk are not read.
struct TableRows {
  const double *p;
  int ks, nk, q;
  __device__ __forceinline__ TableRows(const double *A, int rs, int ks_, int nr, int nk_, int r0, int c, int q_)
      : p(A + (size_t)min(r0 + c, nr - 1) * rs), ks(ks_), nk(nk_), q(q_) {}
};
struct alignas(8) Run4 { double v[4]; };

__device__ __forceinline__ void load_block(double *a, const TableRows &R, int b) {
  const int k = 16 * b + 4 * R.q;
  if (16 * b + 16 <= R.nk && R.ks == 1) {
    const Run4 t = *reinterpret_cast<const Run4 *>(R.p + k);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = t.v[i];
  } else if (16 * b < R.nk) {
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = R.p[(size_t)min(k + i, R.nk - 1) * R.ks];
  }
}

// acc += the block's columns times rows 16 b + 4 q + i of B ([k][kCwLd], LDS,
// zero from nk to the block's end): result row r0 + q + 4 v of chain c in acc[v].
__device__ __forceinline__ void mul_block(v4d &acc, const double *a, int nk, const double *B, int b, int c, int q) {
  if (16 * b < nk) {
    double y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = B[(16 * b + 4 * q + i) * kCwLd + c];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], y[i], acc, 0, 0, 0);
  }
}

struct Half {   // four blocks
  double a[16];
  __device__ __forceinline__ void load(const TableRows &R, int b) {
#pragma unroll
    for (int u = 0; u < 4; ++u) load_block(a + 4 * u, R, b + u);
  }
  __device__ __forceinline__ void mul(v4d &acc, int nk, const double *B, int b, int c, int q) const {
#pragma unroll
    for (int u = 0; u < 4; ++u) mul_block(acc, a + 4 * u, nk, B, b + u, c, q);
  }
};

// The wave's 16 rows of (table) B; h0, h1 hold the table's blocks on entry and
// those of `next` on return (up to 128 columns; the ninth block of a table of
// 129 is read here).
__device__ __forceinline__ v4d table_product(Half &h0, Half &h1, const TableRows &R, const double *B, int c,
                                             const TableRows &next) {
  v4d acc{0.0, 0.0, 0.0, 0.0};
  h0.mul(acc, R.nk, B, 0, c, R.q);
  h0.load(next, 0);
  h1.mul(acc, R.nk, B, 4, c, R.q);
  h1.load(next, 4);
  if (R.nk > 128) {
    double a[4];
    load_block(a, R, 8);
    mul_block(acc, a, R.nk, B, 8, c, R.q);
  }
  return acc;
}

// Forward: the delay at the md sample times t_j = j T_D / md, its transform a_D
// (Eq. det_F_basis), then d_bar = d - S_D a_D (reversed order, zero-padded, as
// k_std_fwd reads it) and c_bar = c - 2 e_D^T a_D + a_D^T Q_D a_D.
__global__ __launch_bounds__(kCwT, 4) void k_std_cw_fwd(StdDev S, const double *__restrict__ x) {
  __shared__ double cst[kCwChains * pt::kCwRows];
  __shared__ double hs[kCwRowsMax * kCwLd];   // the delays, later S_D a_D
  __shared__ double ad[kCwRowsMax * kCwLd];
  __shared__ double cpart[kCwT / 64][kCwChains];
  const int tid = threadIdx.x, w = tid >> 6, c = tid & 15, q = (tid & 63) >> 4;
  const int nb = (S.n_chains + kCwChains - 1) / kCwChains;
  const int pi = xcd_index(blockIdx.x, gridDim.x);
  const int I = pi / nb, c0 = (pi - I * nb) * kCwChains;
  const int nc = min(kCwChains, S.n_chains - c0);
  const int K2 = 2 * S.kd, M = S.md, P = S.P, pp = S.pp;
  const TableRows dft(S.cw_dft, M, 1, K2, M, 16 * w, c, q);
  const TableRows sd(S.cw_sd + (size_t)I * P * K2, K2, 1, P, K2, 16 * w, c, q);
  const TableRows qd(S.cw_qd + (size_t)I * K2 * K2, 1, K2, K2, K2, 16 * w, c, q);   // (symmetric)
  cw_block_constants(S, x, I, c0, nc, cst);
  __syncthreads();
  {
    const pt::CwLane L = cw_lane(cst + c * pt::kCwRows);
    for (int j = tid >> 4; j < kCwRowsMax; j += kCwT / 16)
      hs[j * kCwLd + c] = (c < nc && j < M) ? L.delay<true, false>((double)j * S.td / M).h : 0.0;
  }
  Half h0, h1;
  h0.load(dft, 0);
  h1.load(dft, 4);
  __syncthreads();
  const v4d a = table_product(h0, h1, dft, hs, c, sd);   // a_D
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = 16 * w + q + 4 * v;
    ad[r * kCwLd + c] = r < K2 ? a[v] : 0.0;
  }
  __syncthreads();
  for (int e = tid; e < nc * K2; e += kCwT) {
    const int ch = e / K2, k = e - ch * K2;
    S.cw_ad[((size_t)(c0 + ch) * S.n_psr + I) * K2 + k] = ad[k * kCwLd + ch];
  }
  // S_D a_D, and a_D^T (Q_D a_D - 2 e_D) per chain
  {
    v4d s{0.0, 0.0, 0.0, 0.0};
    if (16 * w < P) {
      s = table_product(h0, h1, sd, ad, c, qd);
    } else {
      h0.load(qd, 0);
      h1.load(qd, 4);
    }
    v4d qa{0.0, 0.0, 0.0, 0.0};
    h0.mul(qa, K2, ad, 0, c, q);
    h1.mul(qa, K2, ad, 4, c, q);
    double part = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * w + q + 4 * v;
      hs[r * kCwLd + c] = s[v];
      if (r < K2) part += a[v] * (qa[v] - 2.0 * S.cw_ed[(size_t)I * K2 + r]);
    }
    part = ln::row_sum_d(part);
    if (q == 0) cpart[w][c] = part;
  }
  __syncthreads();
  for (int e = tid; e < nc * pp; e += kCwT) {
    const int ch = e / pp, r = e - ch * pp;
    S.dbar[((size_t)(c0 + ch) * S.n_psr + I) * pp + r] =
        r < P ? S.dvec[(size_t)I * pp + r] - hs[(P - 1 - r) * kCwLd + ch] : 0.0;
  }
  if (tid < nc) {
    double cb = 0.0;
#pragma unroll
    for (int u = 0; u < kCwT / 64; ++u) cb += cpart[u][tid];
    S.cbar[(size_t)(c0 + tid) * S.n_psr + I] = S.cconst[2 * I] + cb;
  }
}

// dlog p / d a_D = -S_D^T g + beta (e_D - Q_D a_D) with g = dlog p / d d_bar
// (k_std_bwd), then g_h = (transform)^T dlog p / d a_D at the sample times and
// the pulsar's part of dlog p / d theta_cw = sum_j g_h,j dh_j / d theta.
__global__ __launch_bounds__(kCwT, 4) void k_std_cw_bwd(StdDev S, const double *__restrict__ x) {
  __shared__ double cst[kCwChains * pt::kCwRows];
  __shared__ double gb[kCwRowsMax * kCwLd];   // dlog p / d d_bar, later g_h
  __shared__ double ad[kCwRowsMax * kCwLd];   // a_D, later dlog p / d a_D
  const int tid = threadIdx.x, w = tid >> 6, c = tid & 15, q = (tid & 63) >> 4;
  const int nb = (S.n_chains + kCwChains - 1) / kCwChains;
  const int pi = xcd_index(blockIdx.x, gridDim.x);
  const int I = pi / nb, c0 = (pi - I * nb) * kCwChains;
  const int nc = min(kCwChains, S.n_chains - c0);
  const int K2 = 2 * S.kd, M = S.md, P = S.P;
  const TableRows sdt(S.cw_sd + (size_t)I * P * K2, 1, K2, K2, P, 16 * w, c, q);
  const TableRows qd(S.cw_qd + (size_t)I * K2 * K2, 1, K2, K2, K2, 16 * w, c, q);
  const TableRows dft(S.cw_dft, 1, M, M, K2, 16 * w, c, q);
  Half h0, h1;
  h0.load(sdt, 0);
  h1.load(sdt, 4);
  cw_block_constants(S, x, I, c0, nc, cst);
  for (int e = tid; e < kCwChains * kCwRowsMax; e += kCwT) {
    const int ch = e / kCwRowsMax, j = e - ch * kCwRowsMax;
    const size_t ci = (size_t)(c0 + (ch < nc ? ch : 0)) * S.n_psr + I;
    gb[j * kCwLd + ch] = (ch < nc && j < P) ? S.gdbar[ci * P + j] : 0.0;
    ad[j * kCwLd + ch] = (ch < nc && j < K2) ? S.cw_ad[ci * K2 + j] : 0.0;
  }
  __syncthreads();
  {
    const v4d s1 = table_product(h0, h1, sdt, gb, c, qd);
    const v4d s2 = table_product(h0, h1, qd, ad, c, dft);
    __syncthreads();
    const double beta = (c < nc && S.beta) ? S.beta[c0 + c] : 1.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * w + q + 4 * v;
      ad[r * kCwLd + c] = r < K2 ? beta * (S.cw_ed[(size_t)I * K2 + r] - s2[v]) - s1[v] : 0.0;
    }
  }
  __syncthreads();
  // g_h at the sample times (the 129th in a tile of its own)
  {
    v4d gh{0.0, 0.0, 0.0, 0.0};
    h0.mul(gh, K2, ad, 0, c, q);
    h1.mul(gh, K2, ad, 4, c, q);
#pragma unroll
    for (int v = 0; v < 4; ++v) gb[(16 * w + q + 4 * v) * kCwLd + c] = gh[v];
    if (M > 128 && w == 0) {
      const TableRows last(S.cw_dft, 1, M, M, K2, 128, c, q);
      h0.load(last, 0);
      h1.load(last, 4);
      gh = v4d{0.0, 0.0, 0.0, 0.0};
      h0.mul(gh, K2, ad, 0, c, q);
      h1.mul(gh, K2, ad, 4, c, q);
#pragma unroll
      for (int v = 0; v < 4; ++v) gb[(128 + q + 4 * v) * kCwLd + c] = gh[v];
    }
  }
  __syncthreads();
  // the waveform's derivative: chain tid / 32, samples tid % 32 + 32 i, then
  // the 32 lanes of the chain summed in order
  {
    constexpr int LC = kCwT / kCwChains;
    const int ch = tid / LC, lc = tid % LC;
    double out[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (ch < nc) {
      const double *cc = cst + ch * pt::kCwRows;
      const pt::CwLane L = cw_lane(cc);
      double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      for (int j = lc; j < M; j += LC) L.adjoint(L.delay<true, false>((double)j * S.td / M), gb[j * kCwLd + ch], acc);
      // the sky pair through the antenna derivatives, ln 10 for the log10 parameters
      out[0] = -(cc[pt::kCwDfpC] * acc[0] + cc[pt::kCwDfxC] * acc[1]);
      out[1] = -(cc[pt::kCwDfpP] * acc[0] + cc[pt::kCwDfxP] * acc[1]);
      out[2] = ps::kLn10 * acc[2];
      out[3] = ps::kLn10 * acc[3];
      out[4] = acc[4];
      out[5] = acc[5];
      out[6] = acc[6];
      out[7] = ps::kLn10 * acc[7];
    }
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      double t = out[v];
#pragma unroll
      for (int o = LC / 2; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
      out[v] = t;
    }
    if (ch < nc && lc == 0) {
      double *o = S.dcw + ((size_t)(c0 + ch) * S.n_psr + I) * 8;
#pragma unroll
      for (int v = 0; v < 8; ++v) o[v] = out[v];
    }
  }
}

// ---------------------------------------------------------------------------
// Assembly per chain: log p, the hyper-parameter gradient and the status.
// One workgroup of kFinT threads per chain.  Loops over the chain's entries
// issue their loads together; every sum is taken in a fixed order (per-lane
// strides, then fixed shuffle trees and wave partials in wave order).
// ---------------------------------------------------------------------------
constexpr int kFinT = 1024, kFinW = kFinT / 64;

// Sum over the 32 lanes of a half-wave (fixed tree).
__device__ inline double half_sum(double v) {
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__global__ __launch_bounds__(kFinT) void k_std_finalize(StdDev S, const double *x,
                                                         double *__restrict__ logp, double *__restrict__ grad,
                                                         int32_t *__restrict__ status, ps::StdKick kick,
                                                         int has_kick) {
  __shared__ double red[kFinW];
  __shared__ int sb[kFinW][1];
  __shared__ double drho_tot[ps::kMaxRhoK];
  __shared__ double cwp[kFinW][8];
  const int tid = threadIdx.x, c = blockIdx.x, wv = tid >> 6;
  const int n = S.n_psr;
  const double *xc = x + (size_t)c * S.d;
  double *gc = grad + (size_t)c * S.d;
  // Phase one: every load of the input checks, the flags and the log p parts
  // is issued before any is used (fixed batches per thread with clamped
  // in-range addresses, selected when consumed; a remainder loop beyond the
  // batch), then they are combined in the same per-thread order.
  int bad_box = 0, bad_in = 0;
  // the box on theta (two entries a thread per pass)
  constexpr int BB = 2;
  double bxv[BB], blo[BB], bhi[BB];
  {
    const int lt = max(S.n_theta - 1, 0);
#pragma unroll
    for (int u = 0; u < BB; ++u) {
      const int i = min(tid + u * kFinT, lt);
      bxv[u] = S.n_theta > 0 ? xc[i] : 0.0;
      blo[u] = S.n_theta > 0 ? S.prior_lo[i] : 0.0;
      bhi[u] = S.n_theta > 0 ? S.prior_hi[i] : 0.0;
    }
  }
  // finiteness of z (eight entries a thread per pass)
  constexpr int BZ = 8;
  double zv[BZ];
#pragma unroll
  for (int u = 0; u < BZ; ++u) zv[u] = xc[min(S.n_theta + tid + u * kFinT, S.d - 1)];
  // factorisation flags and the log p parts of the pulsars (one a thread)
  int fl = 0;
  double lp = 0.0;
  int f1 = 0, fs = 0, f2 = 0;
  double l0 = 0.0, l1 = 0.0, q0 = 0.0, q1 = 0.0;
  {
    const int i = min(tid, n - 1);
    f1 = S.flag1[(size_t)c * n + i];
    const double *o = S.lik + ((size_t)c * n + i) * 2;
    l0 = o[0];
    l1 = o[1];
  }
  // diagonal prior items: red-only frequencies and DM, or with split
  // coefficients the whole pulsar-noise set (eight a thread per pass; the
  // planner admits no data set without frequencies, so nd >= 1)
  const int kt = S.ka + S.kdm, nd = n * kt;
  constexpr int BD = 8;
  int f3[BD];
  double d0[BD], d1[BD];
#pragma unroll
  for (int u = 0; u < BD; ++u) {
    const int i = min(tid + u * kFinT, nd - 1);
    f3[u] = S.flag3[(size_t)c * nd + i];
    const double *o = S.diag_q + ((size_t)c * nd + i) * 2;
    d0[u] = o[0];
    d1[u] = o[1];
  }
  // the loads that exist only with split coefficients or a common process
  // come last (a wait their branches may take leaves the rest in flight)
  if (S.split) fs = S.flag_s[(size_t)c * 2 * n + min(tid, 2 * n - 1)];
  if (S.nf_gw > 0) {
    const int k = min(tid, S.nf_gw - 1);
    f2 = S.flag2[(size_t)c * S.ka + k];
    const double *oq = S.quad_k + ((size_t)c * S.ka + k) * 2;
    q0 = oq[0];
    q1 = oq[1];
  }
  // d/drho_k in total: the explicit prior part plus the transform's part
  // summed over the pulsars (with split coefficients the pulsars' rho parts
  // are drho_p, and dD_rn holds their kappa parts only), 32 lanes per
  // frequency, pulsars h, h + 32, ... in order
  const int kr = tid >> 5, hr = tid & 31;
  static_assert(4 * 32 >= PTAFS_MAX_PSR, "four passes of 32 lanes cover the pulsars");
  double rv[4], re = 0.0;
  if (S.nf_gw > 0) {
    const double *src = S.split ? S.drho_p : S.dD_rn;
    const int kc = min(kr, S.nf_gw - 1);
#pragma unroll
    for (int m = 0; m < 4; ++m) rv[m] = src[((size_t)c * n + min(hr + 32 * m, n - 1)) * S.ka + kc];
    re = S.drho_e[(size_t)c * S.ka + kc];
  }
  // the box and z checks
#pragma unroll
  for (int u = 0; u < BB; ++u)
    if (tid + u * kFinT < S.n_theta && !(bxv[u] >= blo[u] && bxv[u] <= bhi[u])) bad_box = 1;
  for (int i = tid + BB * kFinT; i < S.n_theta; i += kFinT) {
    const double v = xc[i];
    if (!(v >= S.prior_lo[i] && v <= S.prior_hi[i])) bad_box = 1;
  }
#pragma unroll
  for (int u = 0; u < BZ; ++u)
    if (S.n_theta + tid + u * kFinT < S.d && !isfinite(zv[u])) bad_in = 1;
  for (int i0 = S.n_theta + BZ * kFinT + tid; i0 < S.d; i0 += 4 * kFinT) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = (i0 + u * kFinT < S.d) ? xc[i0 + u * kFinT] : 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (!isfinite(v[u])) bad_in = 1;
  }
  // the CW must not coalesce before the last sample time of its basis
  int bad_cw = 0;
  if (S.has_cw && tid == 0) {
    const double *tc = xc + S.off_cw;
    const double M = exp(ps::kLn10 * tc[2]) * pt::kTsun, w0 = pt::kPi * exp(ps::kLn10 * tc[3]);
    const double K1 = 256.0 / 5.0 * exp((5.0 / 3.0) * log(M * w0)) * w0;
    const double y = K1 * ((double)(S.md - 1) * S.td / S.md);
    bad_cw = !(y < 1.0);
  }
  if (tid < n) {
    fl |= f1;
    lp += l0 + l1;
  }
  if (S.split && tid < 2 * n) fl |= fs;
  if (tid < S.nf_gw) {
    fl |= f2;
    lp += -0.5 * q0 - (n * ps::kLn2Pi + q1);
  }
#pragma unroll
  for (int u = 0; u < BD; ++u) {
    const int i = tid + u * kFinT;
    const int kk = i % kt;
    if (i < nd && (S.split ? (kk < S.nf_rn || kk >= S.ka) : kk >= S.nf_gw)) {
      fl |= f3[u];
      lp += -0.5 * d0[u] - (ps::kLn2Pi + d1[u]);
    }
  }
  for (int i = tid + BD * kFinT; i < nd; i += kFinT) {
    const int kk = i % kt;
    if (S.split ? (kk < S.nf_rn || kk >= S.ka) : kk >= S.nf_gw) {
      fl |= S.flag3[(size_t)c * nd + i];
      const double *o = S.diag_q + ((size_t)c * nd + i) * 2;
      lp += -0.5 * o[0] - (ps::kLn2Pi + o[1]);
    }
  }
  // (d/drho_k: the pulsars' parts summed per frequency)
  if (S.nf_gw > 0) {
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if (kr < S.nf_gw && hr + 32 * m < n) s += rv[m];
    s = half_sum(s);
    if (hr == 0 && kr < S.nf_gw) drho_tot[kr] = re + s;
  }
  // the CW parameters' parts, pulsars in order: lane groups of 8 per wave,
  // then the waves in order
  if (S.has_cw) {
    const int v = tid & 7, I0 = tid >> 3;
    double s = 0.0;
    for (int I = I0; I < n; I += kFinT / 8) s += S.dcw[((size_t)c * n + I) * 8 + v];
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
    if ((tid & 63) < 8) cwp[wv][v] = s;
  }
  __syncthreads();
  // hyper-parameter gradient, 32 lanes per process instance (the common
  // process, then red noise and DM per pulsar), lane k taking frequency k;
  // a lane group's instances it = g, g + 32, ... take their loads together
  {
    constexpr int RB = (1 + 2 * PTAFS_MAX_PSR + kFinT / 32 - 1) / (kFinT / 32);
    const int k = tid & 31, g = tid >> 5, n_it = 1 + 2 * n;
    const int kl = min(k, PTAFS_MAX_HARM - 1);
    double dd[RB], sa[RB], sb2[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int it = g + (kFinT / 32) * r;
      int proc, I, off, K;
      if (it == 0) { proc = 0; I = 0; off = S.off_gw; K = S.nf_gw; }
      else if (it <= n) { proc = 1; I = it - 1; off = S.off_rn + I * S.w_rn; K = S.nf_rn; }
      else { proc = 2; I = min(it - 1 - n, n - 1); off = S.off_dm + I * S.w_dm; K = S.kdm; }
      const bool ok = it < n_it && k < K;
      const int kc = ok ? k : 0;
      dd[r] = 0.0;
      if (ok && proc == 0) dd[r] = drho_tot[kc];
      else if (ok && proc == 1)
        dd[r] = S.dkap_e[((size_t)c * n + I) * S.ka + kc] + S.dD_rn[((size_t)c * n + I) * S.ka + kc];
      else if (ok)
        dd[r] = S.ddm_e[((size_t)c * n + I) * S.kdm + kc] + S.dD_dm[((size_t)c * n + I) * S.kdm + kc];
      // the spectrum's inputs: theta_k (free spectrum) or (log10 A, gamma)
      const int o1 = min(ok ? off + (S.free_spec ? kc : 0) : 0, S.d - 1);
      sa[r] = xc[o1];
      sb2[r] = S.free_spec ? 0.0 : xc[min(o1 + 1, S.d - 1)];
    }
    const double lf = S.lnfy[kl];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int it = g + (kFinT / 32) * r;
      if (it >= n_it) break;
      int off, K;
      if (it == 0) { off = S.off_gw; K = S.nf_gw; }
      else if (it <= n) { off = S.off_rn + (it - 1) * S.w_rn; K = S.nf_rn; }
      else { off = S.off_dm + (it - 1 - n) * S.w_dm; K = S.kdm; }
      if (K == 0) continue;
      double v = 0.0;
      if (k < K) {
        // the spectrum as spec_value forms it
        const double sv = S.free_spec ? exp(ps::kLn10 * sa[r])
                                      : exp(2.0 * ps::kLn10 * sa[r] - sb2[r] * lf + S.pl_c);
        v = sv * dd[r];
      }
      if (S.free_spec) {
        if (k < K) gc[off + k] = ps::kLn10 * v;
      } else {
        const double ga = half_sum(2.0 * ps::kLn10 * v);
        const double gg = half_sum(k < K ? -lf * v : 0.0);
        if (k == 0) {
          gc[off] = ga;
          gc[off + 1] = gg;
        }
      }
    }
  }
  if (S.has_cw && tid < 8) {
    double g = 0.0;
    for (int w = 0; w < kFinW; ++w) g += cwp[w][tid];
    gc[S.off_cw + tid] = g;
  }
  // reduce the flags and log p
  {
    double v = lp;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int bb = __any(bad_box), bi = __any(bad_in), bf = __any(fl != 0), bc = __any(bad_cw);
    if ((tid & 63) == 0) {
      red[wv] = v;
      sb[wv][0] = bb | (bi << 1) | (bf << 2) | (bc << 3);
    }
    __syncthreads();
    // lane i of every wave takes wave i's values, then a second wave
    // reduction (a fixed tree; two registers instead of all waves' values)
    const int ln = tid & 63;
    double t = ln < kFinW ? red[ln] : 0.0;
    int f = ln < kFinW ? sb[ln][0] : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      t += __shfl_xor(t, o, 64);
      f |= __shfl_xor(f, o, 64);
    }
    lp = t;
    bad_box = f & 1;
    bad_in = (f >> 1) & 1;
    fl = (f >> 2) & 1;
    bad_cw = (f >> 3) & 1;
  }
  lp += S.prior_const;
  // output finiteness (the theta entries written above by other threads)
  // and, inside a trajectory, the kick's operands: loaded together, nine
  // entries a thread (every coordinate up to 9216), the rest after
  constexpr int BK = 9;
  double gv[BK], pv[BK], xv[BK], mv[BK];
  double *xw = kick.x + (size_t)c * S.d, *pw = kick.p + (size_t)c * S.d;
#pragma unroll
  for (int u = 0; u < BK; ++u) {
    const int i = min(tid + u * kFinT, S.d - 1);
    gv[u] = gc[i];
    pv[u] = has_kick ? pw[i] : 0.0;
    xv[u] = has_kick ? xw[i] : 0.0;
    mv[u] = (has_kick && kick.inv_mass) ? kick.inv_mass[i] : 1.0;
  }
  int nonfin = !isfinite(lp);
#pragma unroll
  for (int u = 0; u < BK; ++u)
    if (tid + u * kFinT < S.d && !isfinite(gv[u])) nonfin = 1;
  for (int i0 = BK * kFinT + tid; i0 < S.d; i0 += 4 * kFinT) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = (i0 + u * kFinT < S.d) ? gc[i0 + u * kFinT] : 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (!isfinite(v[u])) nonfin = 1;
  }
  nonfin = __syncthreads_or(nonfin);
  int st = PTAFS_ST_OK;
  if (bad_box) st = PTAFS_ST_PRIOR;
  else if (bad_in) st = PTAFS_ST_NONFINITE;
  else if (bad_cw) st = PTAFS_ST_CW;
  else if (fl) st = PTAFS_ST_NOTPD;
  else if (nonfin) st = PTAFS_ST_NONFINITE;
  if (st != PTAFS_ST_OK)
    for (int i = tid; i < S.d; i += kFinT) gc[i] = 0.0;
  if (tid == 0) {
    logp[c] = (st == PTAFS_ST_OK) ? lp : -INFINITY;
    status[c] = st;
  }
  if (has_kick) {
    // inside a trajectory: kick and drift of this chain (the gradient is
    // zero when the status is nonzero)
    if (tid == 0 && kick.n_invalid && st != PTAFS_ST_OK) kick.n_invalid[c] += 1;
#pragma unroll
    for (int u = 0; u < BK; ++u) {
      const int i = tid + u * kFinT;
      if (i < S.d) {
        const double pi = pv[u] + kick.eps * (st != PTAFS_ST_OK ? 0.0 : gv[u]);
        pw[i] = pi;
        xw[i] = xv[u] + kick.eps * mv[u] * pi;
      }
    }
    if (S.d <= BK * kFinT) return;
    __syncthreads();   // every entry of the gradient row is final
    for (int i0 = BK * kFinT + tid; i0 < S.d; i0 += 2 * kFinT) {
      double rg[2], rp[2], rx[2], rm[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int i = i0 + u * kFinT;
        const bool in = i < S.d;
        rg[u] = in ? gc[i] : 0.0;
        rp[u] = in ? pw[i] : 0.0;
        rx[u] = in ? xw[i] : 0.0;
        rm[u] = (in && kick.inv_mass) ? kick.inv_mass[i] : 1.0;
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int i = i0 + u * kFinT;
        if (i < S.d) {
          const double pi = rp[u] + kick.eps * rg[u];
          pw[i] = pi;
          xw[i] = rx[u] + kick.eps * rm[u] * pi;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Split coefficients (App. C, Eqs. separated_post, split_map_a,
// split_standardizing_transform).  The common process and the pulsar noise
// get coefficient sets of their own on the same basis, a = E_G a_G + E_R a_R,
//   a_G = a_hat_G + L_G z_G,  L_G L_G^T = (beta S0_GG + diag rho^-1)^-1,
//   a_R = a_hat_R + L_R z_R,  L_R L_R^T = (beta S0_RR + diag phi_R^-1)^-1,
// and the MAP pair of the joint system is the CURN MAP of the combined
// coefficients split in proportion to the prior variances:
// a_hat_G = rho / D a_hat, a_hat_R = phi_R / D a_hat, D = rho + phi_R (a
// shared row's likelihood sees only the sum, and for a fixed sum the two
// independent Gaussian priors are largest at that split).  k_std_fwd with
// z = 0 gives a_hat; k_split_fac factorises each set; k_split_comb forms
// a_G, a_R, a and the likelihood.  The prior keeps the HD correlations on
// a_G (rho_k Gamma per frequency, Gamma^-1 once per data set) and is
// diagonal on a_R.
// ---------------------------------------------------------------------------

// Set b of pulsar I, chain c: A~ = beta S0_b~ + diag(1 / v~) factorised and
// inverted as the CURN precision is; L_b z_b = X^T z~ and ln det L_b.
template <int T>
__global__ __launch_bounds__(64 * elim_waves<T>(), elim_occ<T>()) void k_split_fac(StdDev S, const double *__restrict__ x,
                                                                              int b) {
  constexpr int W = elim_waves<T>(), pp = 16 * T;
  using E = el::Elim<T, W>;
  __shared__ el::Lds<T, W> L;
  __shared__ double zv[2 * pp], va[pp];
  __shared__ int flag;
  const int tid = el::placed_tid<W>();
  const int pi = xcd_index(blockIdx.x, gridDim.x);
  const int I = pi / S.n_chains, c = pi - I * S.n_chains;
  const double *xc = x + (size_t)c * S.d;
  const double beta = S.beta ? S.beta[c] : 1.0;
  const int PB = b ? S.PR : S.PG;
  const size_t ci = (size_t)c * S.n_psr + I;
  E el(tid);
  load_gram<T>(el, (b ? S.s0r : S.s0g) + (size_t)I * pp * pp);
  const int vt = E::vec_tid(tid);
  if (vt >= 0) {
    bool bad = false;
#pragma unroll
    for (int u = 0; u < (pp + 63) / 64; ++u) {
      const int r = vt + 64 * u;
      if (r >= pp) break;
      zv[2 * r] = (r < PB) ? xc[S.off_z + I * S.pz + (b ? S.PG : 0) + (PB - 1 - r)] : 0.0;
      zv[2 * r + 1] = 0.0;
      if (r >= PB) va[r] = 1.0;
    }
    if (2 * vt < PB) {   // (a lane per frequency)
      const double v = ps::split_var(S, xc, I, b, 2 * vt);
      bad = !(v > 0.0 && isfinite(v));
      const double di = 1.0 / v;
      va[PB - 1 - 2 * vt] = di;
      va[PB - 2 - 2 * vt] = di;
    }
    bad = __any(bad);
    if (vt == 0) flag = bad ? 0 : 1;
  }
  __syncthreads();
  gram_slots<T>(el, beta, va);
  __syncthreads();
  el.template run<0, 0>(L, &flag, nullptr, nullptr, [](int) {});
  double *part = L.row;
  el.xty(part, zv);
  __syncthreads();
  el::store_x(el, (b ? S.xr : S.xg) + ci * (E::NT * 256));
  if (vt < 0) return;
  double part_j = 0.0;
  for (int r = vt; r < PB; r += 64) {
    (b ? S.lzr : S.lzg)[ci * pp + (PB - 1 - r)] = el::xty_sum<T, 2>(part, 0, r);
    part_j += log(L.rs[r]);
  }
  part_j = wave_sum(part_j);
  if (vt == 0) {
    S.jac_s[ci * 2 + b] = part_j;
    S.flag_s[ci * 2 + b] = flag ? 0 : ps::kFlagNotPD;
  }
}

// Per (pulsar, block of 16 chains): a_G, a_R and a from the combined MAP (avec,
// written by k_std_fwd with z = 0) and the sets' L_b z_b; v1 = beta (d - S0 a) and
// beta log L(a) with S0 a formed directly (a is no longer a_hat + L z of one
// factorisation), one matrix product for the block (S0 is read once for 16
// chains); the Jacobian ln det L_G + ln det L_R.  Eight waves, the rows of one
// tile each; thread tid takes row tid % 128 of the chains tid / 128, tid / 128 + 4,
// ... where vectors are read or written, and loads all of them before the first
// is used (with the loads inside the branches of the sets 32 us at 67 pulsars x
// 64 chains, with sixteen waves and two rounds of workgroups 38).
// What bounds it: the vectors (28 MB, 6 us there) and the chain from the prior
// variances to the stores.  Per (pulsar, chain) with S0 read for each it took
// 65 us (7.6 TB/s from L2), now 24.
constexpr int kCombT = 512;

// Spectrum of one process at frequency k from its parameters a (and b).
struct SpecIn { double a, b; };
__device__ __forceinline__ SpecIn spec_load(const StdDev &S, const double *xc, int off, int k, bool in) {
  const int o = !in ? 0 : S.free_spec ? off + k : off;
  return {xc[o], S.free_spec ? 0.0 : xc[o + 1]};
}
__device__ __forceinline__ double spec_eval(const StdDev &S, SpecIn p, double lnfy, bool in) {
  const double e = S.free_spec ? ps::kLn10 * p.a : 2.0 * ps::kLn10 * p.a - p.b * lnfy + S.pl_c;
  return in ? exp(e) : 0.0;
}

__global__ __launch_bounds__(kCombT, 4) void k_split_comb(StdDev S, const double *__restrict__ x) {
  constexpr int NR = 16 * ps::kMaxTiles, G = kCombT / NR, NC = kCwChains / G;
  __shared__ double av[NR * kCwLd];   // a, reversed order, later S0~ a~
  __shared__ double red[kCombT / 64][NC][2];
  const int tid = threadIdx.x, w = tid >> 6;
  const int nb = (S.n_chains + kCwChains - 1) / kCwChains;
  const int pi = xcd_index(blockIdx.x, gridDim.x);
  const int I = pi / nb, c0 = (pi - I * nb) * kCwChains;
  const int nc = min(kCwChains, S.n_chains - c0);
  const int P = S.P, pp = S.pp, j = tid & (NR - 1), g0 = tid / NR;
  const int c16 = tid & 15, q = (tid & 63) >> 4;
  double a[NC], d[NC];
  {
    // row j: the sets it is in, its frequency there, and the set's row (rows past
    // P and chains past nc read the last and write nothing)
    const int jj = min(j, P - 1);
    const bool dm = jj >= 2 * S.ka, in_g = jj < S.PG, in_r = dm || jj < 2 * S.nf_rn;
    const int k = (dm ? jj - 2 * S.ka : jj) >> 1, jr = dm ? jj - 2 * S.ka + 2 * S.nf_rn : jj;
    const int off_r = dm ? S.off_dm + I * S.w_dm : S.off_rn + I * S.w_rn;
    const double lnfy = S.lnfy[k];
    double ah[NC], lg[NC], lr[NC];
    SpecIn pg[NC], pr[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      const int c = c0 + min(g0 + G * u, nc - 1);
      const double *xc = x + (size_t)c * S.d;
      const size_t ci = (size_t)c * S.n_psr + I, vb = ci * pp;
      pg[u] = spec_load(S, xc, S.off_gw, k, in_g);
      pr[u] = spec_load(S, xc, off_r, k, in_r);
      ah[u] = S.avec[vb + jj];
      lg[u] = S.PG ? S.lzg[ci * S.ppg + (in_g ? jj : 0)] : 0.0;
      lr[u] = S.PR ? S.lzr[ci * S.ppr + (in_r ? jr : 0)] : 0.0;
      d[u] = (S.has_cw ? S.dbar + vb : S.dvec + (size_t)I * pp)[P - 1 - jj];
    }
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      const int ch = g0 + G * u;
      const size_t ci = (size_t)(c0 + ch) * S.n_psr + I;
      const double vg = spec_eval(S, pg[u], lnfy, in_g), vr = spec_eval(S, pr[u], lnfy, in_r);
      const double id = 1.0 / (vg + vr);
      const bool on = ch < nc && j < P;
      const double g = in_g ? vg * id * ah[u] + lg[u] : 0.0, r = in_r ? vr * id * ah[u] + lr[u] : 0.0;
      if (on && in_g) S.ag[ci * S.ppg + j] = g;
      if (on && in_r) S.ar[ci * S.ppr + jr] = r;
      a[u] = on ? g + r : 0.0;
      av[(j < P ? P - 1 - j : j) * kCwLd + ch] = a[u];
    }
  }
  const TableRows s0(S.s0 + (size_t)I * pp * pp, pp, 1, pp, pp, 16 * w, c16, q);
  Half h0, h1;
  h0.load(s0, 0);
  h1.load(s0, 4);
  __syncthreads();
  v4d acc{0.0, 0.0, 0.0, 0.0};
  h0.mul(acc, pp, av, 0, c16, q);
  h1.mul(acc, pp, av, 4, c16, q);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) av[(16 * w + q + 4 * v) * kCwLd + c16] = acc[v];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    const int ch = g0 + G * u, c = c0 + ch;
    double pd = 0.0, pq = 0.0;
    if (ch < nc && j < P) {
      const double beta = S.beta ? S.beta[c] : 1.0;
      const size_t vb = ((size_t)c * S.n_psr + I) * pp;
      const double s = av[(P - 1 - j) * kCwLd + ch];
      S.avec[vb + j] = a[u];
      S.v1[vb + (P - 1 - j)] = beta * (d[u] - s);
      pd = a[u] * d[u];
      pq = a[u] * s;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      pd += __shfl_xor(pd, o, 64);
      pq += __shfl_xor(pq, o, 64);
    }
    if ((tid & 63) == 0) {
      red[w][u][0] = pd;
      red[w][u][1] = pq;
    }
  }
  __syncthreads();
  if (tid < nc) {
    const int u = tid / G, w0 = 2 * (tid % G), c = c0 + tid;   // chain tid in the waves w0, w0 + 1
    const double sd = red[w0][u][0] + red[w0 + 1][u][0], sq = red[w0][u][1] + red[w0 + 1][u][1];
    const double beta = S.beta ? S.beta[c] : 1.0;
    const size_t ci = (size_t)c * S.n_psr + I;
    const double *k2 = S.cconst + 2 * I;
    const double cc = S.has_cw ? S.cbar[ci] : k2[0];
    double *o = S.lik + ci * 2;
    o[0] = beta * ((k2[1] - 0.5 * cc) + (sd - 0.5 * sq));
    o[1] = S.jac_s[ci * 2] + S.jac_s[ci * 2 + 1];
  }
}

// Prior of the common set per (frequency k < nf_gw, chain): a_G,k ~ N(0,
// rho_k Gamma) for sin and cos; u = Gamma^-1 a, the quadratic form a^T u /
// rho_k, ln det = N_p ln rho_k + ln det Gamma, -u / rho_k into v2 and the
// explicit derivative (a_s^T u_s + a_c^T u_c) / (2 rho_k^2) - N_p / rho_k.
__global__ __launch_bounds__(256) void k_split_prior_g(StdDev S, const double *__restrict__ x) {
  if (prior_diag_group<256>(S, x, S.n_chains * S.nf_gw)) return;
  __shared__ double as[2][16 * ps::kMaxTiles];
  __shared__ double red[4];
  const int tid = threadIdx.x;
  const int c = blockIdx.x / S.nf_gw, k = blockIdx.x - c * S.nf_gw;
  const int n = S.n_psr;
  const double *xc = x + (size_t)c * S.d;
  const double rho = ps::spec_value(S, xc, 0, 0, k);
  const int i = tid & 127, h = tid >> 7;
  if (i < n) as[h][i] = S.ag[((size_t)c * n + i) * S.ppg + 2 * k + h];
  __syncthreads();
  double part = 0.0;
  if (i < n) {
    double u = 0.0;
    for (int m = 0; m < n; ++m) u = fma(S.gam_inv[(size_t)m * n + i], as[h][m], u);
    part = as[h][i] * u;
    S.v2[((size_t)c * n + i) * S.pp + 2 * k + h] = -u / rho;
  }
  const double q = block_sum(part, red);
  if (tid == 0) {
    double *o = S.quad_k + ((size_t)c * S.ka + k) * 2;
    o[0] = q / rho;
    o[1] = n * log(rho) + S.ldet_gamma;
    S.drho_e[(size_t)c * S.ka + k] = 0.5 * q / (rho * rho) - n / rho;
    S.flag2[(size_t)c * S.ka + k] = (rho > 0.0 && isfinite(rho)) ? 0 : ps::kFlagNotPD;
  }
}

// Adjoint of set b per (pulsar, chain): g = dlog p / d a_b (the likelihood's
// beta (d - S0 a) on the set's rows plus its prior term), dlog p / dz~ = X g~,
// and the set's transform part of dlog p / dv_r, (T_r + Sigma~_rr / 2) / v_r^2
// with T_r and Sigma~_rr as in k_std_bwd (no MAP term: the sets' MAP comes
// from the combined problem).
template <int T>
__global__ __launch_bounds__(64 * AdjX<T>::W, 4) void k_split_bwd(StdDev S, const double *__restrict__ x,
                                                               double *__restrict__ grad, int b) {
  constexpr int pp = 16 * T;
  __shared__ double wp[T * pp], vv[pp], gd[pp];
  __shared__ double2 wz[pp];
  const int tid = threadIdx.x;
  const int pi = (int)gridDim.x - 1 - xcd_index(blockIdx.x, gridDim.x);   // the latest X first
  const int I = pi / S.n_chains, c = pi - I * S.n_chains;
  const double *xc = x + (size_t)c * S.d;
  const int PB = b ? S.PR : S.PG, P = S.P;
  const size_t ci = (size_t)c * S.n_psr + I;
  AdjX<T> X((b ? S.xr : S.xg) + ci * (ps::ntiles(T) * 256), tid);
  const int zo = S.off_z + I * S.pz + (b ? S.PG : 0);
  const int r = tid;
  double zr = 0.0;
  if (r < pp) {
    double g = 0.0;
    if (r < PB) {
      const int j = PB - 1 - r, jc = ps::split_row(S, b, j);
      g = S.v1[ci * S.pp + (P - 1 - jc)] + (b ? S.v2r[ci * pp + j] : S.v2[ci * S.pp + j]);
      (b ? S.gar : S.gag)[ci * pp + j] = g;
      zr = xc[zo + j];
    }
    vv[r] = g;
  }
  __syncthreads();
  X.rows(vv, wp);
  __syncthreads();
  if (r < pp) {
    const double s = AdjX<T>::row_total(wp, r);
    wz[r] = double2{s, zr};
    if (r < PB) grad[(size_t)c * S.d + zo + (PB - 1 - r)] = s;
  }
  __syncthreads();
  X.columns(wz, [&](int col, const ColSum &s) { gd[col] = s.tt + 0.5 * s.ss; });
  __syncthreads();
  if (r < PB) {
    const int j = PB - 1 - r;
    const double v = ps::split_var(S, xc, I, b, j);
    (b ? S.ddr : S.ddg)[ci * pp + j] = gd[r] / (v * v);
  }
}

// Adjoint of the combined MAP per (pulsar, chain) and the chain rule to the
// prior variances.  Upstream of a_hat: g_j = (rho_j g_G,j + phi_j g_R,j) / D_j
// (rho_j = 0 off the common rows, phi_j = 0 off the pulsar-noise rows);
// dlog p / dD_j = a_hat_j (Sigma g)_j / D_j^2 through a_hat, and with
// q_j = a_hat_j / D_j^2 the proportional split adds
//   d/drho_j: phi_j q_j (g_G,j - g_R,j),   d/dphi_j: rho_j q_j (g_R,j - g_G,j);
// each set adds its own transform part.  Rows summed in sin/cos pairs: the
// pulsar's part of dlog p / drho_k (drho_p) and dlog p / dkappa (dD_rn, dD_dm).
// With a CW, dlog p / d d_bar = beta (a + Sigma g).
template <int T>
__global__ __launch_bounds__(64 * AdjX<T>::W, T == 8 ? 3 : 4) void k_split_bwd_c(StdDev S, const double *__restrict__ x) {
  constexpr int pp = 16 * T;
  __shared__ double wp[T * pp], vv[pp], sg[pp], prt[pp], pkt[pp];
  __shared__ double2 wz[pp];
  const int tid = threadIdx.x;
  const int pi = xcd_index(blockIdx.x, gridDim.x);
  const int I = pi / S.n_chains, c = pi - I * S.n_chains;
  const double *xc = x + (size_t)c * S.d;
  const int P = S.P;
  const size_t ci = (size_t)c * S.n_psr + I, vb = ci * pp;
  AdjX<T> X(S.xinv + ci * (ps::ntiles(T) * 256), tid);
  // this thread's row r of X (row j = P - 1 - r of the original order), kept for
  // the chain rule
  const int r = tid, j = P - 1 - r;
  double rho = 0.0, phi = 0.0, gG = 0.0, gR = 0.0, D = 1.0, ah = 0.0;
  int jr = -1;
  if (r < P) {
    D = ps::curn_var(S, xc, I, j);
    ah = S.ahat[vb + r];
    if (j < S.PG) {
      rho = ps::spec_value(S, xc, 0, I, j >> 1);
      gG = S.gag[ci * S.ppg + j];
    }
    if (j < 2 * S.nf_rn || j >= 2 * S.ka) {
      jr = j < 2 * S.nf_rn ? j : j - 2 * S.ka + 2 * S.nf_rn;
      phi = ps::split_var(S, xc, I, 1, jr);
      gR = S.gar[ci * S.ppr + jr];
    }
  }
  if (r < pp) vv[r] = r < P ? (rho * gG + phi * gR) / D : 0.0;
  __syncthreads();
  X.rows(vv, wp);
  __syncthreads();
  if (r < pp) wz[r] = double2{AdjX<T>::row_total(wp, r), 0.0};
  __syncthreads();
  // (Sigma g)~_r = sum_{a >= r} X_ar w~_a
  X.columns(wz, [&](int col, const ColSum &s) { sg[col] = s.sv; });
  __syncthreads();
  if (r < P) {
    const double q = ah / (D * D);
    const double dD = sg[r] * q;
    prt[j] = (j < S.PG) ? dD + phi * q * (gG - gR) + S.ddg[ci * S.ppg + j] : 0.0;
    pkt[j] = (jr >= 0) ? dD + rho * q * (gR - gG) + S.ddr[ci * S.ppr + jr] : 0.0;
    if (S.has_cw) {
      const double beta = S.beta ? S.beta[c] : 1.0;
      S.gdbar[ci * P + j] = beta * (S.avec[vb + j] + sg[r]);
    }
  }
  __syncthreads();
  for (int k = tid; k < S.nf_gw; k += blockDim.x) S.drho_p[ci * S.ka + k] = prt[2 * k] + prt[2 * k + 1];
  for (int k = tid; k < S.nf_rn; k += blockDim.x) S.dD_rn[ci * S.ka + k] = pkt[2 * k] + pkt[2 * k + 1];
  for (int k = tid; k < S.kdm; k += blockDim.x)
    S.dD_dm[ci * S.kdm + k] = pkt[2 * S.ka + 2 * k] + pkt[2 * S.ka + 2 * k + 1];
}

}  // namespace

namespace psk {

#define PS_DISPATCH(TT, KERNEL, WAVES, GRID, ...)                                            \
  switch (TT) {                                                                              \
    case 1: hipLaunchKernelGGL(KERNEL<1>, dim3(GRID), dim3(64 * WAVES(1)), 0, s, __VA_ARGS__); break; \
    case 2: hipLaunchKernelGGL(KERNEL<2>, dim3(GRID), dim3(64 * WAVES(2)), 0, s, __VA_ARGS__); break; \
    case 3: hipLaunchKernelGGL(KERNEL<3>, dim3(GRID), dim3(64 * WAVES(3)), 0, s, __VA_ARGS__); break; \
    case 4: hipLaunchKernelGGL(KERNEL<4>, dim3(GRID), dim3(64 * WAVES(4)), 0, s, __VA_ARGS__); break; \
    case 5: hipLaunchKernelGGL(KERNEL<5>, dim3(GRID), dim3(64 * WAVES(5)), 0, s, __VA_ARGS__); break; \
    case 6: hipLaunchKernelGGL(KERNEL<6>, dim3(GRID), dim3(64 * WAVES(6)), 0, s, __VA_ARGS__); break; \
    case 7: hipLaunchKernelGGL(KERNEL<7>, dim3(GRID), dim3(64 * WAVES(7)), 0, s, __VA_ARGS__); break; \
    case 8: hipLaunchKernelGGL(KERNEL<8>, dim3(GRID), dim3(64 * WAVES(8)), 0, s, __VA_ARGS__); break; \
    default: return hipErrorInvalidValue;                                                    \
  }
#define ELIM_WAVES(T) elim_waves<T>()
#define PRIOR_WAVES(T) prior_waves<T>()
#define ADJ_WAVES(T) AdjX<T>::W

hipError_t launch_std_cw_fwd(const StdDev &S, const double *x, hipStream_t s) {
  const int grid = ((S.n_chains + kCwChains - 1) / kCwChains) * S.n_psr;
  if (grid == 0 || !S.has_cw) return hipSuccess;
  hipLaunchKernelGGL(k_std_cw_fwd, dim3(grid), dim3(kCwT), 0, s, S, x);
  return hipGetLastError();
}

hipError_t launch_std_cw_bwd(const StdDev &S, const double *x, hipStream_t s) {
  const int grid = ((S.n_chains + kCwChains - 1) / kCwChains) * S.n_psr;
  if (grid == 0 || !S.has_cw) return hipSuccess;
  hipLaunchKernelGGL(k_std_cw_bwd, dim3(grid), dim3(kCwT), 0, s, S, x);
  return hipGetLastError();
}

hipError_t launch_std_fwd(const StdDev &S, const double *x, hipStream_t s) {
  const int grid = S.n_chains * S.n_psr;
  if (grid == 0) return hipSuccess;
  PS_DISPATCH(S.tp, k_std_fwd, ELIM_WAVES, grid, S, x);
  return hipGetLastError();
}

hipError_t launch_std_prior(const StdDev &S, const double *x, hipStream_t s) {
  const size_t items =
      (size_t)S.n_chains * S.n_psr * ((S.split ? S.nf_rn : S.ka - S.nf_gw) + S.kdm);
  if (S.n_chains > 0 && S.nf_gw > 0) {   // the diagonal items after the dense problems
    const int nd = S.n_chains * S.nf_gw, nth = S.split || S.tg > 4 ? 256 : 64;
    static_assert(prior_waves<4>() == 1 && prior_waves<5>() == 4, "threads of a workgroup by tiles");
    const int grid = nd + (int)((items + nth - 1) / nth);
    if (S.split) hipLaunchKernelGGL(k_split_prior_g, dim3(grid), dim3(256), 0, s, S, x);
    else PS_DISPATCH(S.tg, k_std_prior_dense, PRIOR_WAVES, grid, S, x);
  } else if (items) {
    hipLaunchKernelGGL(k_std_prior_diag, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, S, x);
  }
  return hipGetLastError();
}

hipError_t launch_std_bwd(const StdDev &S, const double *x, double *grad, hipStream_t s) {
  const int grid = S.n_chains * S.n_psr;
  if (grid == 0) return hipSuccess;
  PS_DISPATCH(S.tp, k_std_bwd, ADJ_WAVES, grid, S, x, grad);
  return hipGetLastError();
}

// Split coefficients: the two sets' factorisations, then a_G, a_R, a and the
// likelihood (after launch_std_fwd, which gives the combined MAP).
hipError_t launch_split_fwd(const StdDev &S, const double *x, hipStream_t s) {
  const int grid = S.n_chains * S.n_psr;
  if (grid == 0 || !S.split) return hipSuccess;
  PS_DISPATCH(S.tpg, k_split_fac, ELIM_WAVES, grid, S, x, 0);
  PS_DISPATCH(S.tpr, k_split_fac, ELIM_WAVES, grid, S, x, 1);
  hipLaunchKernelGGL(k_split_comb, dim3(((S.n_chains + kCwChains - 1) / kCwChains) * S.n_psr), dim3(kCombT), 0, s, S, x);
  return hipGetLastError();
}

// Split coefficients: the sets' adjoints, then the combined MAP's and the
// chain rule (in place of launch_std_bwd).
hipError_t launch_split_bwd(const StdDev &S, const double *x, double *grad, hipStream_t s) {
  const int grid = S.n_chains * S.n_psr;
  if (grid == 0 || !S.split) return hipSuccess;
  PS_DISPATCH(S.tpg, k_split_bwd, ADJ_WAVES, grid, S, x, grad, 0);
  PS_DISPATCH(S.tpr, k_split_bwd, ADJ_WAVES, grid, S, x, grad, 1);
  PS_DISPATCH(S.tp, k_split_bwd_c, ADJ_WAVES, grid, S, x);
  return hipGetLastError();
}

hipError_t launch_std_finalize(const StdDev &S, const double *x, double *logp, double *grad,
                               int32_t *status, hipStream_t s, const ps::StdKick *kick) {
  if (S.n_chains == 0) return hipSuccess;
  const ps::StdKick k = kick ? *kick : ps::StdKick{};
  hipLaunchKernelGGL(k_std_finalize, dim3(S.n_chains), dim3(kFinT), 0, s, S, x, logp, grad, status, k,
                     kick ? 1 : 0);
  return hipGetLastError();
}

}  // namespace psk
