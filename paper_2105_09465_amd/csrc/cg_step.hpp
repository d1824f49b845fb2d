// End of a conjugate-gradient iteration of one column (cg.hip, cg_small.hip).
#pragma once

#include "common.hpp"
#include "internal.hpp"

namespace gpl {

// alpha = rr / pAp, or the breakdown code: 1 for p.Ap <= 0 or an alpha that is not
// finite, 2 for a p.Ap that is not.
struct ColumnAlpha {
  double alpha;
  int bad;
};
__device__ __forceinline__ ColumnAlpha cg_alpha(double rr, double pap) {
  const double a = rr / pap;
  const bool ok = (pap > 0.0) && isfinite(a);
  return ColumnAlpha{ok ? a : 0.0, ok ? 0 : (isfinite(pap) ? 1 : 2)};
}

// From the state st before the iteration, alpha, the breakdown code and the new r.r:
// beta, the next state, and whether P is updated; `record` writes the Lanczos
// coefficients.
struct ColumnStep {
  ColState next;
  double beta;
  int go;
};
__device__ __forceinline__ ColumnStep cg_step(const ColState& st, double alpha, int bad, double rr_new, int c,
                                              const double* bb, double tol, int max_iter, int fixed_iters,
                                              int n_lanczos, double* ab, bool record) {
  const double beta = rr_new / st.rr;
  ColState nx;
  nx.alpha = alpha;
  nx.bad = 0;
  nx.iters = st.iters;
  nx.rr = st.rr;
  nx.status = GPL_CG_CONVERGED;
  nx.active = 0;
  int go = 0;
  if (bad) {
    nx.status = bad == 1 ? GPL_CG_BREAKDOWN : GPL_CG_NONFINITE;
  } else if (!isfinite(rr_new) || !isfinite(beta)) {
    nx.status = GPL_CG_NONFINITE;
    nx.iters = st.iters + 1;
  } else {
    go = 1;
    nx.rr = rr_new;
    nx.iters = st.iters + 1;
    if (record && st.iters < n_lanczos) {
      double* e = ab + ((size_t)c * n_lanczos + st.iters) * 2;
      e[0] = alpha;
      e[1] = beta;
    }
    if (fixed_iters > 0) {
      nx.active = nx.iters < fixed_iters;
    } else if (sqrt(rr_new) <= tol * sqrt(bb[c])) {
      nx.active = 0;
    } else if (nx.iters >= max_iter) {
      nx.status = GPL_CG_MAXITER;
    } else {
      nx.active = 1;
    }
  }
  return ColumnStep{nx, beta, go};
}

// The vector part of an iteration on a small image, one workgroup per column: the
// partial rows of the product's launch to B^T P of the next iteration in the
// product's buffers (cg_small.hip).
struct CgColumn {
  int n, ss, nrhs, ntiles;
  float sigma2, amp2;
  Taps taps;
  TilePlan plan;
  ProdBufs bufs;
  RhsOut rhs;
  float *X, *R, *P;
  int ldx, ldv;
  const double* bb;
  double tol;
  int max_iter, fixed_iters, n_lanczos;
  double* ab;
};
bool cg_column_fits(int n, int ss, int r);
// st_in, st_out: the states before and after; active: counts of active columns, read
// ([0]), added to ([1], cleared an iteration before) and cleared ([2]).
int cg_column_launch(const CgColumn& C, const ColState* st_in, ColState* st_out, const int* active_in,
                     int* active_out, int* active_next, hipStream_t stream);

}  // namespace gpl
