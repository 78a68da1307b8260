// Dense per-frequency prior covariance of arrays of 81 to 128 pulsars (six to
// eight 16-row tiles) on FP64 matrix cores, four waves per (frequency, chain).
//
// Forward (Sec. IV.A, Eqs. HD, prior_cov; Sec. II.B, Eq. standardizing_transform
// with mu = 0): C = chol(rho_k Gamma + diag kappa_.k) by the register elimination
// of elim_dev.h without its inverse, a_.k,{sin,cos} = C z_.k,{sin,cos} on the
// way, C kept for the adjoint.
//
// Backward, with abar from the TOA pass: v_c = C^T abar_c, dz_c = v_c - z_c, and
// with W = C^-1, M = W chol(Gamma), P = Phi(sum_c v_c z_c^T)
//   d/dkappa_I = w_I^T P w_I,  d/drho = sum_I m_I^T P m_I.
// The block columns of W (and of M) are independent: W_IJ = -W_II sum_{J<=K<I}
// C_IK W_KJ, so a wave takes the columns J and NT - 1 - J (nine tiles of eight
// rows, whatever J), with C and then W in LDS, and there is no barrier inside
// a column.  Two problems fit a compute unit (80 KB of LDS each).
//
// What bounds them: the chain of one problem (16 chains x 30 frequencies are
// 480 problems for 256 compute units), in the forward the eight diagonal tiles
// one after the other.  Per launch at 120 pulsars, 16 chains and 30 frequencies:
// forward 40 us, adjoint 45.  A thread per row of L took 411 us, a thread per
// column of C^-1 (rows of C as scalar loads) 373, each with a launch for the
// diagonal frequencies (9 and 6 us) beside it; one wave per problem, at 110
// pulsars, 84 and 68.
//
// Layouts of a tile X (lane l = c + 16 q, item v or slice s), as in k_cholt's
// adjoint: A(X): X[pi(c)][4q + s], B(X): X[4q + v][c].
#include "common.h"
#include "elim_dev.h"
#include "quad_dev.h"
#include "spec_dev.h"

namespace {

using ln::mfma4;
using ln::v4d;
using pt::Dev;
using pt::pk;
using ps::tix;

constexpr int kW = 4;       // waves per problem
constexpr int kPerCu = 2;   // problems a compute unit (one wave of each a SIMD)

// the factor C of a problem: tile-major with row-major tiles up to seven
// tiles, packed row-major beyond (chol_store_doubles)
template <int NT>
struct FactorOut {
  static constexpr bool kOn = true;
  double *dst;
  int n, c, q;
  __device__ inline void below(int I, int J, const v4d &l) {   // rows q + 4 v of C_IJ
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * I + q + 4 * v;
      if (NT <= pt::kTileStoreNT) dst[tix(I, J) * 256 + (q + 4 * v) * 16 + c] = l[v];
      else if (r < n) dst[pk(r, 16 * J + c)] = l[v];
    }
  }
  __device__ inline void diagonal(int J, const v4d &lt) {      // columns q + 4 v of C_JJ
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * J + c, k = 16 * J + q + 4 * v;
      if (NT <= pt::kTileStoreNT) dst[tix(J, J) * 256 + 16 * c + q + 4 * v] = lt[v];
      else if (r < n && k <= r) dst[pk(r, k)] = lt[v];
    }
  }
};

// grid: nf_gw c_pad problems, and the diagonal-frequency workgroups after them
// (FIRST: before)
template <int NT, bool FIRST>
__global__ __launch_bounds__(64 * kW, kPerCu) void k_cholw_fwd(Dev D, const double *__restrict__ x, int n_dense) {
  static_assert(64 * kW == 256, "the diagonal-frequency work runs on 256 threads");
  const int prob = FIRST ? (int)(blockIdx.x - (gridDim.x - n_dense)) : (int)blockIdx.x;
  if (FIRST ? prob < 0 : prob >= n_dense) {
    const pt::spec_split sp(D, gridDim.x - n_dense, D.c_pad, false);
    for (int it = FIRST ? blockIdx.x : prob - n_dense; it < sp.nb * sp.ns; it += sp.G) {
      const int b = it / sp.ns, s = it - b * sp.ns;
      pt::spec_fwd_cb(D, x, b * pt::kCB, sp.k_lo(s), sp.k_lo(s + 1), s, sp.ns);
      __syncthreads();
    }
    return;
  }
  constexpr int NP = 16 * NT;
  static_assert(NP <= 64 * kW, "a thread per row");
  using E = el::Elim<NT, kW>;
  __shared__ el::Lds<NT, kW> L;
  __shared__ double bv[2 * NP], tv[2 * NP], kb[NP];   // C z, z (sin, cos), kappa
  __shared__ int fail;
  const int k0 = prob % D.nf_gw, c = prob / D.nf_gw;
  const int tid = el::placed_tid<kW>();
  const int n = D.n_psr;
  const size_t cp = D.c_pad;
  const int rs = pt::harm_row(k0 + 1, 0), rc = pt::harm_row(k0 + 1, 1);
  int32_t *flag = D.flag_dense + (size_t)c * D.nf_gw + k0;
  const double *xc = x + (size_t)(c < D.n_chains ? c : 0) * D.d;
  E el(tid);
  // every load before the first use: the Gamma tiles (column-major: a slot's
  // rows of block C and columns of block I), the row's spectrum and z, the box
#pragma unroll
  for (int s = 0; s < E::NS; ++s) {
    const double *g = D.gam_tile + (el.has(s) ? tix(el.tile_i(s), el.tile_c(s)) : 0) * 256 + el.lane;
#pragma unroll
    for (int v = 0; v < 4; ++v) el.a[s][v] = g[64 * v];
  }
  const int rr = tid < n ? tid : n - 1;
  const double kl = xc[D.off_rn + 2 * rr], kg = xc[D.off_rn + 2 * rr + 1];
  const double *z = xc + D.off_z + (size_t)rr * 2 * D.ka + 2 * k0;
  const double z0 = z[0], z1 = z[1];
  const double rho = pt::powerlaw_k(D, k0, xc[D.off_gw], xc[D.off_gw + 1]);
  const bool inbox = c < D.n_chains && pt::theta_in_box_wave(D, xc);   // the same in every wave
  double *out_s = D.coef_rn + ((size_t)tid * D.rows_rn + rs) * cp + c;
  double *out_c = D.coef_rn + ((size_t)tid * D.rows_rn + rc) * cp + c;
  if (!inbox) {
    if (tid < n) {
      *out_s = 0.0;
      *out_c = 0.0;
    }
    if (tid == 0) *flag = 0;
    return;
  }
  if (tid < NP) {
    const bool real = tid < n;
    kb[tid] = !real ? 1.0 : k0 < D.nf_rn ? pt::powerlaw_k(D, k0, kl, kg) : 0.0;
    tv[2 * tid] = real ? z0 : 0.0;
    tv[2 * tid + 1] = real ? z1 : 0.0;
    bv[2 * tid] = bv[2 * tid + 1] = 0.0;
  }
  if (tid == 0) fail = 1;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < E::NS; ++s) {
    el.a[s] *= -rho;
    if (el.tile_i(s) == el.tile_c(s)) {
      const double kv = kb[16 * el.tile_i(s) + el.c];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (el.q + 4 * v == el.c) el.a[s][v] -= kv;
    }
  }
  FactorOut<NT> out{D.lstore + ((size_t)c * D.nf_gw + k0) * pt::chol_store_doubles(n), n, el.c, el.q};
  el.template run<0, 2, false>(L, &fail, bv, tv, [](int) {}, out);
  const bool pd = fail != 0;
  if (tid < n) {
    *out_s = pd ? bv[2 * tid] + L.lzd[2 * tid] : 0.0;
    *out_c = pd ? bv[2 * tid + 1] + L.lzd[2 * tid + 1] : 0.0;
  }
  if (tid == 0) *flag = pd ? 0 : pt::kFlagNotPD;
}

// ---------------------------------------------------------------------------
// Backward: grid nf_gw n_chains problems, and the diagonal-frequency workgroups
// after or before them.
// ---------------------------------------------------------------------------

// element (r, c) of an LDS tile: 16 lanes that read a row or a column hit 16 banks
__device__ inline int at(int r, int c) { return (r << 4) + (c ^ r); }
__device__ inline v4d ld_a(const double *t, int pc, int q) {   // A(X)
  return v4d{t[at(pc, 4 * q)], t[at(pc, 4 * q + 1)], t[at(pc, 4 * q + 2)], t[at(pc, 4 * q + 3)]};
}
__device__ inline v4d ld_b(const double *t, int c, int q) {    // B(X)
  return v4d{t[at(4 * q, c)], t[at(4 * q + 1, c)], t[at(4 * q + 2, c)], t[at(4 * q + 3, c)]};
}
__device__ inline void st_b(double *t, int c, int q, const v4d &v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) t[at(4 * q + i, c)] = v[i];
}

template <int NT, bool FIRST>
__global__ __launch_bounds__(64 * kW, kPerCu) void k_cholw_bwd(Dev D, const double *__restrict__ x,
                                                          double *__restrict__ grad,
                                                          const double *__restrict__ lst,
                                                          const double *__restrict__ gch,
                                                          const double *__restrict__ bar, int n_dense) {
  const int prob = FIRST ? (int)(blockIdx.x - (gridDim.x - n_dense)) : (int)blockIdx.x;
  if (FIRST ? prob < 0 : prob >= n_dense) {
    const pt::spec_split sp(D, gridDim.x - n_dense, D.n_chains, true);
    for (int it = FIRST ? blockIdx.x : prob - n_dense; it < sp.nb * sp.ns; it += sp.G) {
      const int b = it / sp.ns, s = it - b * sp.ns;
      pt::spec_bwd_cb(D, x, grad, b * pt::kCB, sp.k_lo(s), sp.k_lo(s + 1), s, sp.ns);
      __syncthreads();
    }
    return;
  }
  constexpr int NP = 16 * NT, NTILE = ps::ntiles(NT), NS = (NTILE + kW - 1) / kW, N2 = NT / 2;
  __shared__ double tl[NTILE][256];                    // C, then W
  __shared__ double vz[NP][4];                         // v_sin, v_cos, z_sin, z_cos
  __shared__ double ab[NP][2];
  __shared__ double drw[kW];
  __shared__ int nbw[kW];
  const int k0 = prob % D.nf_gw, c = prob / D.nf_gw;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, c16 = l & 15, q = l >> 4;
  const int pc = qf::pi16(c16);
  const int n = D.n_psr;
  const int kmax = max(D.ka, D.nf_dm);
  const size_t cp = D.c_pad;
  const int rs = pt::harm_row(k0 + 1, 0), rc = pt::harm_row(k0 + 1, 1);
  const int K2 = 2 * D.ka;
  const double *xc = x + (size_t)c * D.d;
  double *gz = grad + (size_t)c * D.d + D.off_z + 2 * k0;
  double *drn = pt::drn_at(D, c, 0, k0);   // pulsar I at drn[2 ka I]
  const size_t dI = 2 * (size_t)D.ka;
  double *dth = D.dth_k + ((size_t)c * D.ka + k0) * 2;
  const int fl0 = D.flag_k[(size_t)c * kmax + k0] | D.flag_dense[(size_t)c * D.nf_gw + k0];
  int32_t *fout = D.flag_out + (size_t)c * (kmax + pt::kSpecSeg) + k0;
  if (D.st_pre[c] != 0 || fl0 != 0) {
    for (int I = tid; I < n; I += 64 * kW) {
      gz[(size_t)I * K2] = 0.0;
      gz[(size_t)I * K2 + 1] = 0.0;
      drn[dI * I] = 0.0;
      drn[dI * I + 1] = 0.0;
    }
    if (tid == 0) {
      dth[0] = 0.0;
      dth[1] = 0.0;
      *fout = 0;
    }
    return;
  }
  // ---- C (the padding an identity), abar and z into LDS
  const double *Cb = lst + ((size_t)c * D.nf_gw + k0) * pt::chol_store_doubles(n);
  {
    double t[NS][4];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int tt = s * kW + w;
      if (tt >= NTILE) continue;
      int I = 0;
#pragma unroll
      for (int k = 1; k < NT; ++k) I += tt >= tix(k, 0);
      const int J = tt - tix(I, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * I + q + 4 * v, k = 16 * J + c16;
        if (NT <= pt::kTileStoreNT) t[s][v] = Cb[tt * 256 + (q + 4 * v) * 16 + c16];
        else t[s][v] = r < n && k <= r ? Cb[pk(r, k)] : r == k ? 1.0 : 0.0;
      }
    }
    if (tid < NP) {
      double as = 0.0, ac = 0.0, zs = 0.0, zc = 0.0;
      if (tid < n) {
        as = bar[((size_t)tid * D.rows_rn + rs) * cp + c];
        ac = bar[((size_t)tid * D.rows_rn + rc) * cp + c];
        zs = xc[D.off_z + (size_t)tid * K2 + 2 * k0];
        zc = xc[D.off_z + (size_t)tid * K2 + 2 * k0 + 1];
      }
      ab[tid][0] = as;
      ab[tid][1] = ac;
      vz[tid][2] = zs;
      vz[tid][3] = zc;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (s * kW + w >= NTILE) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) tl[s * kW + w][at(q + 4 * v, c16)] = t[s][v];
    }
  }
  __syncthreads();
  // ---- waves 0 and 1: inverses of the diagonal tiles, lane row q taking tile
  //      4 w + q, column c16 by forward substitution (kept in registers until C
  //      is read); waves 2 and 3: v_c = C^T abar_c, block columns in turn
  double xs[16];
  const int Jd = 4 * w + q;
  if (w < 2) {
    if (Jd < NT) {
      const double *T = tl[tix(Jd, Jd)];
      double rdg[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) rdg[r] = ln::rcp_nr(T[at(r, r)]);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        __builtin_amdgcn_sched_barrier(0);   // bound the live LDS reads to one row
        double s = (r == c16) ? 1.0 : 0.0;
#pragma unroll
        for (int m = 0; m < r; ++m) s -= T[at(r, m)] * xs[m];
        xs[r] = s * rdg[r];
      }
    }
  } else {
    for (int J = w - 2; J < NT; J += 2) {
      double ss = 0.0, sc = 0.0;
      for (int K = J; K < NT; ++K) {
        const v4d e = ld_b(tl[tix(K, J)], c16, q);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          ss += e[v] * ab[16 * K + 4 * q + v][0];
          sc += e[v] * ab[16 * K + 4 * q + v][1];
        }
      }
      ss = ln::row_sum_d(ss);
      sc = ln::row_sum_d(sc);
      if (q == 0) {
        vz[16 * J + c16][0] = ss;
        vz[16 * J + c16][1] = sc;
      }
    }
  }
  __syncthreads();
  if (w < 2 && Jd < NT) {
#pragma unroll
    for (int r = 0; r < 16; ++r) tl[tix(Jd, Jd)][at(r, c16)] = xs[r];
  }
  __syncthreads();
  // ---- W = C^-1, block columns J1 and J2 of this wave in registers, and their
  //      d/dkappa quadratic forms.  (With an odd number of tiles the middle
  //      column has no partner, with six the last wave has no columns.)
  const int J1 = w, J2 = NT - 1 - w;
  const bool on1 = J1 <= J2, on2 = J1 < J2;
  v4d W1[NT], W2[N2];
  double dk1 = 0.0, dk2 = 0.0;
  auto column = [&](int J, auto &Wc, double &dk) {
    constexpr int NW = sizeof(Wc) / sizeof(v4d);
    Wc[0] = ld_b(tl[tix(J, J)], c16, q);
#pragma unroll
    for (int i = 1; i < NW; ++i) {
      if (J + i >= NT) break;
      v4d U{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < i; ++k) U = mfma4(ld_a(tl[tix(J + i, J + k)], pc, q), Wc[k], U);
      Wc[i] = mfma4(-ld_a(tl[tix(J + i, J + i)], pc, q), U, v4d{0.0, 0.0, 0.0, 0.0});
    }
    qf::ScanState st{0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      if (J + i >= NT) break;
      qf::scan_tile(Wc[i], 16 * (J + i), vz, st, q);
    }
    dk = ln::row_sum_d(st.q);
  };
  if (on1) column(J1, W1, dk1);
  if (on2) column(J2, W2, dk2);
  __syncthreads();   // every read of C done
  auto store = [&](int J, auto &Wc) {
    constexpr int NW = sizeof(Wc) / sizeof(v4d);
#pragma unroll
    for (int i = 1; i < NW; ++i)
      if (J + i < NT) st_b(tl[tix(J + i, J)], c16, q, Wc[i]);
  };
  if (on1) store(J1, W1);
  if (on2) store(J2, W2);
  __syncthreads();
  // ---- d/drho: M = W G, the same block columns, and their quadratic forms
  double dr = 0.0;
  auto mcolumn = [&](int J, auto &G) {
    constexpr int NW = sizeof(G) / sizeof(v4d);
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      if (J + i >= NT) break;
      const double *gt = gch + tix(J + i, J) * 256 + 64 * q + c16;
      G[i] = v4d{gt[0], gt[16], gt[32], gt[48]};
    }
    qf::ScanState st{0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      if (J + i >= NT) break;
      v4d Mt{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k <= i; ++k) Mt = mfma4(ld_a(tl[tix(J + i, J + k)], pc, q), G[k], Mt);
      qf::scan_tile(Mt, 16 * (J + i), vz, st, q);
    }
    dr += st.q;
  };
  if (on1) mcolumn(J1, W1);   // (W's registers take the columns of G)
  if (on2) mcolumn(J2, W2);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) dr += __shfl_xor(dr, o, 64);
  // ---- outputs of the pulsars of the wave's block columns, and d/drho
  const double lnfy = D.lnfy[k0];
  bool fin = true;
  auto put = [&](int J, double dk) {
    const int I = 16 * J + c16;
    if (q != 0 || I >= n) return;
    const double g0 = vz[I][0] - vz[I][2], g1 = vz[I][1] - vz[I][3];
    gz[(size_t)I * K2] = g0;
    gz[(size_t)I * K2 + 1] = g1;
    const double kap = k0 < D.nf_rn ? pt::powerlaw_k(D, k0, xc[D.off_rn + 2 * I], xc[D.off_rn + 2 * I + 1]) : 0.0;
    const double d0 = dk * kap * 2.0 * pt::kLn10, d1 = dk * kap * (-lnfy);
    drn[dI * I] = d0;
    drn[dI * I + 1] = d1;
    fin = fin && isfinite(g0) && isfinite(g1) && isfinite(d0) && isfinite(d1);
  };
  if (on1) put(J1, dk1);
  if (on2) put(J2, dk2);
  const int nbad = __popcll(__ballot(!fin));
  if (l == 0) {
    drw[w] = dr;
    nbw[w] = nbad;
  }
  __syncthreads();
  if (tid == 0) {
    const double rho = pt::powerlaw_k(D, k0, xc[D.off_gw], xc[D.off_gw + 1]);
    const double d = (drw[0] + drw[1]) + (drw[2] + drw[3]);
    dth[0] = d * rho * 2.0 * pt::kLn10;
    dth[1] = d * rho * (-lnfy);
    const int nb = (nbw[0] + nbw[1]) + (nbw[2] + nbw[3]);
    *fout = (nb || !isfinite(dth[0]) || !isfinite(dth[1])) ? pt::kFlagOutNonfinite : 0;
  }
}

// Diagonal-frequency workgroups beside dense problems that fill the device: they go
// first, about one a compute unit.  Beside fewer they go last, on what the dense
// ones leave free (spec_groups_fwd, spec_groups); beside more than one round they
// would start there when the dense ones end, a few long workgroups at the end of the
// launch.  96 pulsars, 14 common and 30 diagonal frequencies with DM, 48 and 256
// chains: forward 54 and 253 us with them last, 50 and 169 first, adjoint 107 and
// 328, 49 and 204.
inline bool fills(const Dev &D, int np) { return np >= kPerCu * D.n_cu; }
inline int groups_first(const Dev &D, int chains, int max_seg) {
  const int nb = (chains + pt::kCB - 1) / pt::kCB, kmax = max(D.ka, D.nf_dm);
  return nb * max(1, min(min(kmax, max_seg), D.n_cu / nb));
}

template <int NT>
hipError_t launch_fwd_t(const Dev &D, const double *x, hipStream_t s) {
  const int np = D.nf_gw * D.c_pad;
  if (fills(D, np))
    hipLaunchKernelGGL((k_cholw_fwd<NT, true>), dim3(np + groups_first(D, D.c_pad, PTAFS_MAX_HARM)), dim3(64 * kW), 0,
                       s, D, x, np);
  else
    hipLaunchKernelGGL((k_cholw_fwd<NT, false>), dim3(np + pt::spec_groups_fwd(D, np, D.c_pad)), dim3(64 * kW), 0, s, D,
                       x, np);
  return hipGetLastError();
}

template <int NT>
hipError_t launch_bwd_t(const Dev &D, const double *x, double *grad, hipStream_t s) {
  const int np = D.nf_gw * D.n_chains;
  if (fills(D, np))
    hipLaunchKernelGGL((k_cholw_bwd<NT, true>), dim3(np + groups_first(D, D.n_chains, pt::kSpecSeg)), dim3(64 * kW), 0,
                       s, D, x, grad, (const double *)D.lstore, D.gtile, (const double *)D.bar_rn, np);
  else
    hipLaunchKernelGGL((k_cholw_bwd<NT, false>), dim3(np + pt::spec_groups(D, np, D.n_chains, kPerCu)), dim3(64 * kW),
                       0, s, D, x, grad, (const double *)D.lstore, D.gtile, (const double *)D.bar_rn, np);
  return hipGetLastError();
}

}  // namespace

namespace ptk {

hipError_t launch_cholw_fwd(const pt::Dev &D, const double *x, hipStream_t s) {
  switch (pt::chol_tiles(D.n_psr)) {
    case 6: return launch_fwd_t<6>(D, x, s);
    case 7: return launch_fwd_t<7>(D, x, s);
    case 8: return launch_fwd_t<8>(D, x, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_cholw_bwd(const pt::Dev &D, const double *x, double *grad, hipStream_t s) {
  switch (pt::chol_tiles(D.n_psr)) {
    case 6: return launch_bwd_t<6>(D, x, grad, s);
    case 7: return launch_bwd_t<7>(D, x, grad, s);
    case 8: return launch_bwd_t<8>(D, x, grad, s);
  }
  return hipErrorInvalidValue;
}

// Spectral stages: the dense frequencies with the diagonal-frequency work in
// the same launch, or that work alone where no frequency is dense.
hipError_t launch_spectral_fwd(const pt::Dev &D, const double *x, hipStream_t s) {
  if (D.c_pad == 0) return hipSuccess;
  if (D.nf_gw == 0) return launch_spec_fwd(D, x, s);
  return pt::chol_tiles(D.n_psr) <= pt::kTileMaxNT ? launch_cholt_fwd(D, x, s) : launch_cholw_fwd(D, x, s);
}

hipError_t launch_spectral_bwd(const pt::Dev &D, const double *x, double *grad, hipStream_t s) {
  if (D.n_chains == 0) return hipSuccess;
  if (D.nf_gw == 0) return launch_spec_bwd(D, x, grad, s);
  return pt::chol_tiles(D.n_psr) <= pt::kTileMaxNT ? launch_cholt_bwd(D, x, grad, s)
                                                   : launch_cholw_bwd(D, x, grad, s);
}

}  // namespace ptk
