// What follows a reduction on the device: the Gram solves of Lemma 4.1, the
// curvature and the truncated CG's tests, from the sums (PostOp, kernels.h).
#pragma once

#include "common.h"
#include "kernels.h"

namespace gpe {

// Apply a post-operation.  sum: the nq sums; st: the caller's copy of res[0..64),
// which put() keeps current beside res itself (thread 0 only; every value it
// needs was fetched in parallel before).
__device__ inline void finalize_post(const double* sum, int nq, double* st, double* res, int post, int F, double* gram,
                              const double* gin) {
  const int K = 2 * F + 1;
  auto put = [&](int k, double v) {
    st[k] = v;
    res[k] = v;
  };
  if (post == POST_GRAD) {
    // Gram system of Lemma 4.1 (proof) with the measured u^T u, u^T G u, u^T G^2 u
    double a11 = 0, a12 = 0, a22 = 0, r1 = 0, r2 = 0, e = sum[0];
    for (int i = 0; i < K; ++i) {
      double xg = sum[1 + i];
      for (int k = 1 + 2 * K + i; k < nq; k += K) {   // kinetic sums of the axes kept apart
        xg += sum[k];
        e += 0.5 * sum[k];
      }
      const double l = F - i, nrm = sum[1 + K + i];
      a11 += nrm;
      a12 += l * nrm;
      a22 += l * l * nrm;
      r1 += xg;
      r2 += l * xg;
      put(1 + i, xg);
      put(1 + K + i, nrm);
      if (gram) gram[i] = nrm;
    }
    const double det = a11 * a22 - a12 * a12;
    put(0, e);
    put(1 + 2 * K, (a22 * r1 - a12 * r2) / det);
    put(2 + 2 * K, (a11 * r2 - a12 * r1) / det);
  } else if (post == POST_ENERGY) {
    double e = sum[0];
    for (int k = 1; k < nq; ++k) e += 0.5 * sum[k];
    put(0, e);
  } else if (post == POST_HVP_AB) {
    double a11 = 0, a12 = 0, a22 = 0;
    for (int i = 0; i < K; ++i) {
      const double l = F - i;
      a11 += gin[i];
      a12 += l * gin[i];
      a22 += l * l * gin[i];
    }
    const double det = a11 * a22 - a12 * a12;
    put(32, (a22 * sum[0] - a12 * sum[1]) / det);
    put(33, (a11 * sum[1] - a12 * sum[0]) / det);
  } else if (post == POST_HVP_KAPPA || post == POST_HVP_KAPPA_E || post == POST_CG_KAPPA) {
    double zlz = 0.0;
    for (int k = 6; k < nq; ++k) zlz += sum[k];
    const double kappa = post == POST_HVP_KAPPA_E ? sum[4] + zlz : sum[4] + zlz - st[32] * sum[2] - st[33] * sum[3];
    const double pp = sum[5];
    put(34, kappa);
    put(35, pp);
    if (post == POST_CG_KAPPA) {
      const int it = (int)st[CG_IT];   // iterations done before this one
      put(CG_IT, (double)(it + 1));
      if (!(kappa > st[CG_EPS] * pp)) {   // curvature stop (a NaN stops too)
        put(CG_KAPPA, kappa);
        put(CG_PP, pp);
        put(CG_REASON, CG_STOP_CURVATURE);
        put(CG_CURV, 1.0);
        put(CG_DONE, 1.0);
      } else {
        put(CG_ALPHA, st[cg_rr_slot(it)] / kappa);
      }
    }
  } else if (post == POST_CG_STEP) {
    const double rr = sum[0];
    const int it = (int)st[CG_IT];   // iterations done, this one included
    if (sqrt(rr) <= st[CG_TOL]) {
      put(CG_REASON, CG_STOP_RESIDUAL);
      put(CG_DONE, 1.0);
    } else {
      put(CG_BETA, rr / st[cg_rr_slot(it - 1)]);
      put(cg_rr_slot(it), rr);
      if (st[CG_IT] >= st[CG_MAXIT]) {
        put(CG_REASON, CG_STOP_CAP);
        put(CG_DONE, 1.0);
      }
    }
  }
}

}  // namespace gpe
