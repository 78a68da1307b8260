// Quadratic forms x^T P x with the semiseparable P = Phi(sum_c v_c z_c^T) down the
// columns of 16-row tiles (the adjoint of a Cholesky factor), on the layout
// that the adjoints' matrix products leave: lane c + 16 q, item v holds row
// 4 q + v of column c.
#pragma once

#include "lane_dev.h"

namespace qf {

using ln::v4d;
using ln::xor16_d;
using ln::xor32_d;

// row of the A operand's lane c, so that a result's lane row q holds the
// consecutive rows 4 q .. 4 q + 3
__device__ inline int pi16(int c) { return 4 * (c & 3) + (c >> 2); }

struct ScanState {
  double rs, rc, q;   // running column sums of z x (sin, cos) and the quadratic form
};

// One 16-row tile of 16 columns (B layout: item v of lane group q is row
// row0 + 4q + v) added to the column quadratic forms x^T P x; vr[v] holds
// (v_sin, v_cos, z_sin, z_cos) of row row0 + 4q + v.
__device__ inline void scan_rows(const v4d &X, const double (&vr)[4][4], ScanState &st, int q) {
  double ls = 0.0, lc = 0.0, part = 0.0, sa = 0.0, ca = 0.0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const double x = X[v];
    const double bs = vr[v][2] * x, bc = vr[v][3] * x;
    const double as = vr[v][0] * x, ac = vr[v][1] * x;
    part += as * (ls + 0.5 * bs) + ac * (lc + 0.5 * bc);
    ls += bs;
    lc += bc;
    sa += as;
    ca += ac;
  }
  // inclusive prefix of the lane sums over the four lane groups of a column
  // and their total, by the row swaps: with t the partner row's sum, the
  // pair total is p = x + t, the prefix x (+ t on odd rows) (+ the other
  // half's pair total on rows 2 and 3), the total p + that
  const double ts1 = xor16_d(ls, q), tc1 = xor16_d(lc, q);
  const double ps = ls + ts1, pc2 = lc + tc1;
  const double os = xor32_d(ps, q), oc = xor32_d(pc2, q);
  double is = (q & 1) ? ps : ls, ic = (q & 1) ? pc2 : lc;
  if (q >= 2) {
    is += os;
    ic += oc;
  }
  const double ts = ps + os, tc = pc2 + oc;
  st.q += part + (st.rs + (is - ls)) * sa + (st.rc + (ic - lc)) * ca;
  st.rs += ts;
  st.rc += tc;
}

// this lane's rows of v and z for the row tile at row0
__device__ inline void load_rows(const double (*vz)[4], int row0, int q, double (&vr)[4][4]) {
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int k = 0; k < 4; ++k) vr[v][k] = vz[row0 + 4 * q + v][k];
}

__device__ inline void scan_tile(const v4d &X, int row0, const double (*vz)[4], ScanState &st,
                                 int q) {
  double vr[4][4];
  load_rows(vz, row0, q, vr);
  scan_rows(X, vr, st, q);
}

}  // namespace qf
