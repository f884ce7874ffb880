// C ABI entry points (include/gpe.h) and the device operations they are
// built from.  Host code only: every kernel is launched through kernels.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>

#include "common.h"
#include "retract_scalar.h"
#include "runtime.h"

static std::string g_create_error;

namespace gpe {

gpe_status fail(gpe_handle* h, gpe_status s, const std::string& msg) {
  if (h) h->err = msg;
  else g_create_error = msg;
  return s;
}

gpe_status hip_fail(gpe_handle* h, hipError_t e, const char* where) {
  std::string m = std::string("HIP error '") + hipGetErrorString(e) + "' in " + where;
  return fail(h, e == hipErrorOutOfMemory ? GPE_ENOMEM : GPE_EHIP, m);
}

const char* const kKernelNames[KK_COUNT] = {"lap_axis_x", "lap_axis_y", "lap_axis_z", "hvp_xpass",
                                            "pw_grad", "finalize", "project", "comp_norms",
                                            "scale_comps", "vector_ops"};

hipEvent_t timing_event(gpe_handle* h) {
  if (!h->event_pool.empty()) {
    hipEvent_t e = h->event_pool.back();
    h->event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  (void)hipEventCreate(&e);
  return e;
}

gpe_status alloc_field(gpe_handle* h, void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    return fail(h, GPE_ENOMEM, "device allocation of " + std::to_string(bytes) + " bytes failed");
  }
  return GPE_OK;
}

template <typename T>
gpe_status laplacian(gpe_handle* h, const void* in, void* out) {
  for (int a = 0; a < h->dim; ++a) GPE_KT(h, KK_LAP_X + a, lap_axis<T>(h->ax[a], in, a == 0 ? nullptr : out, out, h->F, h->npts, h->st));
  return GPE_OK;
}
template gpe_status laplacian<double>(gpe_handle*, const void*, void*);
template gpe_status laplacian<float>(gpe_handle*, const void*, void*);

gpe_status finalize_enq(gpe_handle* h, int nblk, int nq, int post, double* gram) {
  SlotCounts nb;
  for (int q = 0; q < kMaxQ; ++q) nb.nb[q] = nblk;
  GPE_KT(h, KK_FINALIZE,
         finalize(h->part, nblk, nb, nq, h->res, post, h->F, gram, h->ticket, nullptr, h->hres, h->st));
  return GPE_OK;
}

gpe_status fetch(gpe_handle* h) {
  GPE_HIP(h, hipStreamSynchronize(h->st));   // (the finalize stored its results in hres)
  return GPE_OK;
}

static gpe_status finite(gpe_handle* h, const double* v, int n, const char* what) {
  for (int i = 0; i < n; ++i)
    if (!std::isfinite(v[i])) return fail(h, GPE_ENUMERIC, std::string("NaN or Inf in ") + what);
  return GPE_OK;
}

// The energy at X and, with G, the gradient (Sec. 3).  GRAD_EUCLID: G and the
// multipliers of its projection; GRAD_RIEM: G projected (Lemma 4.1), the
// multipliers staying on the device in between; GRAD_POINT: G = L X, with the
// gradient's sums all the same, X copied to the set point (and its c64 copy),
// the last axis storing G in c64 for a mixed handle.  norm: ||G||^2 into
// res[kResNorm] (always with GRAD_RIEM).
//
// The last axis pass of GRAD_RIEM needs every kinetic sum before it starts, its
// own axis' included: a pass that only reads X and sums comes first (1 field),
// in place of a projection that reads X and G and writes G after it (3 fields).
enum GradKind { GRAD_EUCLID = 0, GRAD_RIEM, GRAD_POINT };
static gpe_status grad_enq(gpe_handle* h, const void* X, void* G, double* gram, GradKind kind, bool norm) {
  const int K = h->K, last = h->dim - 1;
  const bool riem = kind == GRAD_RIEM, point = kind == GRAD_POINT;
  const bool mixed_point = point && h->prec == GPE_MIXED;
  norm = norm || riem;
  if (h->dim == 1) {   // one row: one workgroup does it all
    auto one = [&](auto f) {
      return grad_one<f()>(h->ax[0], X, h->V64, G, point ? h->Xp : nullptr, mixed_point ? h->Xp32 : nullptr, h->pw,
                           point, riem, norm, G ? gram : nullptr, h->res, h->hres, h->st);
    };
    GPE_KT(h, KK_PW_GRAD,
           h->F == 1 ? one(std::integral_constant<int, 1>{}) : h->F == 2 ? one(std::integral_constant<int, 2>{})
                                                                         : one(std::integral_constant<int, 3>{}));
    return GPE_OK;
  }
  int nbx = 0, tpc[3] = {0, 0, 0};
  const int first = G ? 1 + 2 * K : 1;   // slot of the first kinetic sum kept apart
  // axes of which only the sums are wanted, in the x pass' launch where they can be
  auto sum_only = [&](int a) { return !G || (riem && a == last); };
  auto rides = [&](int a) { return sum_only(a) && h->ax[a].n == h->ax[0].n; };
  // (their slots lie past the axis passes', which leave norms in the slot after their own)
  auto kin_slot = [&](int a) { return rides(a) ? first + last + a : first + a - 1; };
  SumAxes sums;
  for (int a = 1; a <= last; ++a)
    if (rides(a)) {
      sums.inner[sums.n] = h->ax[a].inner;
      sums.lamc[sums.n] = h->ax[a].lamc;
      sums.slot[sums.n++] = kin_slot(a);
    }
  auto gx = [&](auto f) {
    return grad_xpass<f()>(h->ax[0], h->npts, X, h->V64, G, point ? h->Xp : nullptr, mixed_point ? h->Xp32 : nullptr,
                           h->pw, point, h->part, h->pstride, &nbx, &sums, h->st);
  };
  GPE_KT(h, KK_PW_GRAD,
         h->F == 1 ? gx(std::integral_constant<int, 1>{}) : h->F == 2 ? gx(std::integral_constant<int, 2>{})
                                                                      : gx(std::integral_constant<int, 3>{}));
  for (int a = 1; a <= last; ++a) {
    if (rides(a)) {
      tpc[a] = sums.tpc;
      continue;
    }
    GPE_KT(h, KK_LAP_X + a,
           grad_axis(h->ax[a], sum_only(a), X, G, G, mixed_point && a == last ? h->LX32 : nullptr, h->F,
                     h->npts, nullptr, nullptr, h->part, h->pstride, first + a - 1, &tpc[a], h->st));
  }
  const size_t ps = h->pstride;
  SlotSegs s;
  auto add = [&](size_t off, int n) {
    s.off[s.nq] = (int)off;
    s.nb[s.nq++] = n;
  };
  for (int q = 0; q < first; ++q) add(q * ps, nbx);
  for (int a = 1; a <= last; ++a) {
    if (!G) add(kin_slot(a) * ps, K * tpc[a]);
    for (int i = 0; G && i < K; ++i) add(kin_slot(a) * ps + (size_t)i * tpc[a], tpc[a]);
  }
  GPE_KT(h, KK_FINALIZE,
         finalize_segs(h->part, s, h->part + (kMaxQ - 1) * ps, h->res, G ? POST_GRAD : POST_ENERGY, h->F,
                       G ? gram : nullptr, h->ticket, norm ? nullptr : h->hres, h->st));
  if (!norm) return GPE_OK;
  if (riem)
    GPE_KT(h, KK_LAP_X + last,
           grad_axis(h->ax[last], false, X, G, G, nullptr, h->F, h->npts, X, h->res + 1 + 2 * K, h->part, ps,
                     first + last - 1, &tpc[last], h->st));
  SlotSegs sn;
  sn.nq = 1;
  sn.off[0] = (int)((first + last) * ps);   // the slot after the last axis' sums
  sn.nb[0] = K * tpc[last];
  GPE_KT(h, KK_FINALIZE,
         finalize_segs(h->part, sn, h->res + kResNorm, h->res, POST_NONE, h->F, nullptr, h->ticket, h->hres, h->st));
  return GPE_OK;
}

gpe_status eval_enq(gpe_handle* h, const void* X, void* G, double* gram) {
  return grad_enq(h, X, G, gram, GRAD_EUCLID, false);
}

gpe_status eval_read(gpe_handle* h, bool grad, double* E, double* ag, double* bg) {
  const int nq = 1 + 2 * h->K;
  const double* r = h->hres;
  // the reductions first; the multipliers after the degeneracy test (a
  // singular Gram system gives NaN multipliers, which is GPE_EDEGEN)
  GPE_TRY(finite(h, r, grad ? nq : 1, "the energy or gradient"));
  if (grad) {
    double a11 = 0, a12 = 0, a22 = 0;
    for (int i = 0; i < h->K; ++i) {
      const double l = h->F - i;
      a11 += r[1 + h->K + i];
      a12 += l * r[1 + h->K + i];
      a22 += l * l * r[1 + h->K + i];
    }
    if (!(a11 * a22 - a12 * a12 > 0))
      return fail(h, GPE_EDEGEN, "degenerate point: u^T Gamma^2 u u^T u - (u^T Gamma u)^2 <= 0");
    GPE_TRY(finite(h, r + nq, 2, "the gradient's multipliers"));
    if (ag) *ag = r[nq];
    if (bg) *bg = r[nq + 1];
  }
  if (E) *E = r[0];
  return GPE_OK;
}

gpe_status pgrad_enq(gpe_handle* h, const void* X, const void* G, void* gR, double ag, double bg) {
  GPE_KT(h, KK_PROJECT,
         launch_single(ProjArgs<double, double, true>{X, G, gR, nullptr, ag, bg, h->part, h->npts, h->F}, h->nblk,
                       h->st));
  return finalize_enq(h, h->nblk, 1, POST_NONE, nullptr);
}

gpe_status pgrad_read(gpe_handle* h, double* gnorm) {
  GPE_TRY(finite(h, h->hres, 1, "the gradient norm"));
  if (gnorm) *gnorm = std::sqrt(h->hres[0]);
  return GPE_OK;
}

gpe_status project_grad(gpe_handle* h, const void* X, const void* G, void* gR, double ag, double bg,
                        double* gnorm) {
  GPE_TRY(pgrad_enq(h, X, G, gR, ag, bg));
  GPE_TRY(fetch(h));
  return pgrad_read(h, gnorm);
}

// cg: one iteration of the device-resident truncated CG (the launches are
// skipped once the CG has stopped, and the last finalize runs its tests).
// kappa: form <Z, HZ> and ||Z||^2 (res[34..35]) in a last finalize; gpe_hvp
// without scalar outputs skips that launch.
template <typename T>
static gpe_status hvp_t(gpe_handle* h, const void* Z, void* HZ, bool riem, const PwParams& p, bool cg,
                        bool kappa) {
  const void* Xw = sizeof(T) == 8 ? h->Xp : h->Xp32;
  const void* Yw = sizeof(T) == 8 ? h->LX64 : h->LX32;
  const T* Vw = reinterpret_cast<const T*>(sizeof(T) == 8 ? (const void*)h->V64 : (const void*)h->V32);
  const double* skip = cg ? h->res + CG_DONE : nullptr;
  const int post = cg ? POST_CG_KAPPA : !kappa ? POST_NONE : riem ? POST_HVP_KAPPA : POST_HVP_KAPPA_E;
  if (h->dim == 1) {   // one row: one workgroup does it all
    GPE_KT(h, KK_HVP_XPASS,
           hvp_one<T>(h->F, h->ax[0], Xw, Z, riem ? Yw : nullptr, Vw, HZ, p, h->gram_pt, h->res,
                      kappa && !cg ? h->hres : nullptr, post, riem, skip, h->st));
    return GPE_OK;
  }
  SlotCounts nb;
  for (int q = 0; q < kMaxQ; ++q) nb.nb[q] = 0;
  int nbx = 0;
  GPE_KT(h, KK_HVP_XPASS,
         hvp_xpass<T>(h->F, h->ax[0], h->npts, Xw, Z, riem ? Yw : nullptr, Vw, HZ, p, h->part, h->pstride, &nbx, h->xvar, skip, h->st));
  for (int q = 0; q < 7; ++q) nb.nb[q] = nbx;
  double* coef = h->res + 32;
  // Projection coefficients (Lemma 4.1) from the x pass's partials: with few
  // rows every workgroup of the last axis pass forms them itself; in 3D
  // otherwise one extra workgroup of the y pass does; else a finalize.
  const bool ab_local = riem && h->npts / (size_t)h->n[0] <= (size_t)kAbLocalMax;
  const bool ab_ypass = riem && !ab_local && h->dim == 3;
  if (riem && !ab_local && !ab_ypass)
    GPE_KT(h, KK_FINALIZE,
           finalize(h->part, h->pstride, nb, 7, h->res, POST_HVP_AB, h->F, h->gram_pt, h->ticket, skip, nullptr,
                    h->st));
  int nq = 7;
  for (int a = 1; a < h->dim; ++a) {
    const bool proj = riem && a == h->dim - 1;
    AbSrc ab, fin;
    if (proj && ab_local) ab = AbSrc{h->part, h->pstride, nbx, h->gram_pt, h->res};
    if (a == 1 && ab_ypass) fin = AbSrc{h->part, h->pstride, nbx, h->gram_pt, h->res};
    GPE_KT(h, KK_LAP_X + a,
           lap_axis_ex<T>(h->ax[a], Z, HZ, HZ, h->F, h->npts, proj ? Xw : nullptr, coef, h->part, h->pstride, 6 + a,
                          &nb.nb[6 + a], skip, a == 1, ab.part ? &ab : nullptr, fin.part ? &fin : nullptr, h->st));
    nq = 7 + a;
  }
  if (post == POST_NONE) return GPE_OK;
  GPE_KT(h, KK_FINALIZE, finalize(h->part, h->pstride, nb, nq, h->res, post, h->F, h->gram_pt, h->ticket, skip,
                                  cg ? nullptr : h->hres, h->st));
  return GPE_OK;
}

// Pick the fused x pass's rows-per-workgroup by timing each variant on the
// handle's own grid.  The fields hold pseudo-random values rather than zeros:
// the cost does not depend on the values, but the power drawn (and so the
// clock the chip sustains) does.
template <typename T>
static gpe_status tune_xpass_t(gpe_handle* h) {
  const int nv = xpass_variants(h->n[0]);
  if (nv <= 1 || h->dim == 1) return GPE_OK;   // (a 1D grid runs whole in one workgroup)
  if (h->npts <= kUntimedPoints) {
    h->xvar = 2;
    return GPE_OK;
  }
  // three distinct fields for X, Z, LX (aliasing them would hide memory traffic)
  void* A = sizeof(T) == 8 ? h->T64 : h->T32;
  void* Bz = sizeof(T) == 8 ? h->Xp : h->Xp32;
  void* C = sizeof(T) == 8 ? h->LX64 : h->LX32;
  void* Wt = h->Gp;                                // scratch output (c128, large enough)
  const T* Vw = reinterpret_cast<const T*>(sizeof(T) == 8 ? (const void*)h->V64 : (const void*)h->V32);
  unsigned seed = 1;
  for (void* b : {A, Bz, C})
    GPE_HIP(h, launch_single(FillArgs<T>{b, h->nel, seed++}, elementwise_blocks(h->nel), h->st));
  hipEvent_t e0, e1;
  GPE_HIP(h, hipEventCreate(&e0));
  GPE_HIP(h, hipEventCreate(&e1));
  float best = 1e30f;
  int bestv = 1;
  for (int v = 0; v < nv; ++v) {
    int nb = 0;
    GPE_HIP(h, hvp_xpass<T>(h->F, h->ax[0], h->npts, A, Bz, C, Vw, Wt, h->pw, h->part, h->pstride, &nb, v, nullptr,
                            h->st));
    float tmin = 1e30f;
    for (int rep = 0; rep < 3; ++rep) {
      GPE_HIP(h, hipEventRecord(e0, h->st));
      GPE_HIP(h, hvp_xpass<T>(h->F, h->ax[0], h->npts, A, Bz, C, Vw, Wt, h->pw, h->part, h->pstride, &nb, v,
                              nullptr, h->st));
      GPE_HIP(h, hipEventRecord(e1, h->st));
      GPE_HIP(h, hipEventSynchronize(e1));
      float ms = 0.f;
      GPE_HIP(h, hipEventElapsedTime(&ms, e0, e1));
      tmin = std::fmin(tmin, ms);
    }
    h->xvar_us[v] = 1e3f * tmin;
    if (tmin < best) {
      best = tmin;
      bestv = v;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  h->xvar = bestv;
  return GPE_OK;
}

gpe_status tune_xpass(gpe_handle* h) {
  return h->prec == GPE_FP64 ? tune_xpass_t<double>(h) : tune_xpass_t<float>(h);
}

PwParams hvp_params(const gpe_handle* h, bool riem, double sigma) {
  PwParams p = h->pw;
  for (int i = 0; i < 7; ++i) p.zc[i] = (riem && i < h->K) ? sigma - h->alpha_g - h->beta_g * (h->F - i) : 0.0;
  return p;
}

gpe_status hvp_enq(gpe_handle* h, const void* Z, void* HZ, bool riem, double sigma, bool cg, bool kappa) {
  if (!h->has_point) return fail(h, GPE_EINVAL, "gpe_hvp before gpe_set_point");
  if (cg && !riem) return fail(h, GPE_EINVAL, "the device-resident CG takes the Riemannian HVP");
  const PwParams p = hvp_params(h, riem, sigma);
  if (!work32(h)) return hvp_t<double>(h, Z, HZ, riem, p, cg, kappa);
  return hvp_t<float>(h, Z, HZ, riem, p, cg, kappa);
}

gpe_status hvp_read(gpe_handle* h, double* kappa, double* zz) {
  GPE_TRY(finite(h, h->hres + 34, 2, "the Hessian-vector product"));
  if (kappa) *kappa = h->hres[34];
  if (zz) *zz = h->hres[35];
  return GPE_OK;
}

gpe_status hvp(gpe_handle* h, const void* Z, void* HZ, bool riem, double sigma, double* kappa, double* zz) {
  GPE_TRY(hvp_enq(h, Z, HZ, riem, sigma, false, kappa || zz));
  if (!kappa && !zz) return GPE_OK;
  GPE_TRY(fetch(h));
  return hvp_read(h, kappa, zz);
}

gpe_status norms_enq(gpe_handle* h, const void* u, const void* xi, bool xi32) {
  if (xi32)
    GPE_KT(h, KK_NORMS, (comp_norms<double, float>(h->K, u, xi, h->part, comp_blocks(h->npts), h->npts, h->st)));
  else
    GPE_KT(h, KK_NORMS, (comp_norms<double, double>(h->K, u, xi, h->part, comp_blocks(h->npts), h->npts, h->st)));
  return finalize_enq(h, comp_blocks(h->npts), xi ? 3 * h->K : h->K, POST_NONE, nullptr);
}

RgbbArgs rgbb_args(const gpe_handle* h, const void* z, const void* gz, const void* u, const void* gu, void* out,
                   double ag, double bg) {
  return RgbbArgs{z, gz, u, gu, out, ag, bg, h->part, h->npts, h->K};
}

// Sums 0 .. 3K-1 per component; the last two over every component (consecutive slots).
SlotSegs rgbb_segs(const gpe_handle* h) {
  const int K = h->K, nbc = comp_blocks(h->npts);
  SlotSegs s;
  s.nq = 3 * K + 2;
  for (int q = 0; q < s.nq; ++q) {
    const int first = q < 3 * K ? q : (q == 3 * K ? 3 * K : 4 * K);
    s.off[q] = first * nbc;
    s.nb[q] = q < 3 * K ? nbc : K * nbc;
  }
  return s;
}

gpe_status rgbb_enq(gpe_handle* h, const void* z, const void* gz, const void* u, const void* gu, void* out, double ag,
                    double bg) {
  GPE_KT(h, KK_PROJECT,
         launch_single(rgbb_args(h, z, gz, u, gu, out, ag, bg), h->K * comp_blocks(h->npts), h->st));
  GPE_KT(h, KK_FINALIZE, finalize_segs(h->part, rgbb_segs(h), h->res, h->res, POST_NONE, h->F, nullptr, h->ticket,
                                       h->hres, h->st));
  return GPE_OK;
}

gpe_status rgbb_read(gpe_handle* h, RetractNorms* rn, double* gnorm, double* sv, double* vv) {
  GPE_TRY(norms_read(h, true, rn));
  GPE_TRY(finite(h, h->hres + 3 * h->K, 2, "the Barzilai-Borwein products"));
  double g2 = 0.0;
  for (int i = 0; i < h->K; ++i) g2 += rn->xx[i];
  *gnorm = std::sqrt(g2);
  *sv = h->hres[3 * h->K];
  *vv = h->hres[3 * h->K + 1];
  return GPE_OK;
}

gpe_status norms_read(gpe_handle* h, bool has_xi, RetractNorms* rn) {
  const int K = h->K;
  GPE_TRY(finite(h, h->hres, has_xi ? 3 * K : K, "the component norms"));
  for (int i = 0; i < K; ++i) {
    rn->uu[i] = h->hres[i];
    rn->ux[i] = has_xi ? h->hres[K + i] : 0.0;
    rn->xx[i] = has_xi ? h->hres[2 * K + i] : 0.0;
  }
  return GPE_OK;
}

gpe_status retract_norms(gpe_handle* h, const void* u, const void* xi, bool xi32, RetractNorms* rn) {
  GPE_TRY(norms_enq(h, u, xi, xi32));
  GPE_TRY(fetch(h));
  return norms_read(h, xi != nullptr, rn);
}

gpe_status retraction_sigma(gpe_handle* h, const double* a, int kind, double* sig) {
  int r;
  switch (kind) {
    case GPE_R1_PROJECTIVE: r = sigma_projective(h->F, h->M, a, sig); break;
    case GPE_R2_ORTHOGONAL: r = sigma_orthogonal(h->F, h->M, a, sig); break;
    case GPE_R3_CLOSED: r = sigma_closed(h->F, h->M, a, sig); break;
    default: return fail(h, GPE_EINVAL, "unknown retraction kind");
  }
  if (r != SIGMA_OK)
    return fail(h, GPE_EDOMAIN, kind == GPE_R3_CLOSED ? "retraction argument outside S"
                                                      : "retraction argument outside Omega");
  return GPE_OK;
}

gpe_status proj_coeffs(gpe_handle* h, const RetractNorms& rn, double* alpha, double* beta) {
  double a11 = 0, a12 = 0, a22 = 0, r1 = 0, r2 = 0;
  for (int i = 0; i < h->K; ++i) {
    const double l = h->F - i;
    a11 += rn.uu[i];
    a12 += l * rn.uu[i];
    a22 += l * l * rn.uu[i];
    r1 += rn.ux[i];
    r2 += l * rn.ux[i];
  }
  const double det = a11 * a22 - a12 * a12;
  if (!(det > 0)) return fail(h, GPE_EDEGEN, "degenerate Gram system in the projection");
  *alpha = (a22 * r1 - a12 * r2) / det;
  *beta = (a11 * r2 - a12 * r1) / det;
  return GPE_OK;
}

gpe_status retract_sigma_at(gpe_handle* h, const RetractNorms& rn, double t, int kind, double* sig) {
  double a[7];
  for (int i = 0; i < h->K; ++i) {
    a[i] = rn.uu[i] + 2.0 * t * rn.ux[i] + t * t * rn.xx[i];   // ||u_i + t xi_i||^2
    if (a[i] < 0) a[i] = 0;
  }
  return retraction_sigma(h, a, kind, sig);
}

gpe_status retract_apply(gpe_handle* h, const RetractNorms& rn, const void* u, const void* xi, bool xi32, double t,
                         int kind, void* out) {
  double sig[7];
  GPE_TRY(retract_sigma_at(h, rn, t, kind, sig));
  if (xi32)
    GPE_KT(h, KK_SCALE, (scale_comps<double, float, double>(h->K, u, xi, t, sig, out, h->npts, h->st)));
  else
    GPE_KT(h, KK_SCALE, (scale_comps<double, double, double>(h->K, u, xi, t, sig, out, h->npts, h->st)));
  return GPE_OK;
}

gpe_status dot_enq(gpe_handle* h, const void* a, bool a32, const void* b, bool b32, size_t n) {
  if (!a32 && !b32) GPE_KT(h, KK_VECTOR, (dot<double, double>(a, b, h->part, h->nblk, n, h->st)));
  else if (a32 && b32) GPE_KT(h, KK_VECTOR, (dot<float, float>(a, b, h->part, h->nblk, n, h->st)));
  else if (!a32 && b32) GPE_KT(h, KK_VECTOR, (dot<double, float>(a, b, h->part, h->nblk, n, h->st)));
  else GPE_KT(h, KK_VECTOR, (dot<double, float>(b, a, h->part, h->nblk, n, h->st)));
  return finalize_enq(h, h->nblk, 1, POST_NONE, nullptr);
}

gpe_status dot_read(gpe_handle* h, double* out) {
  GPE_TRY(finite(h, h->hres, 1, "an inner product"));
  *out = h->hres[0];
  return GPE_OK;
}

gpe_status cg_init_enq(gpe_handle* h, double tol, double eps, int maxit) {
  GPE_KT(h, KK_VECTOR, launch_single(CgInitArgs{h->res, tol, eps, maxit}, 1, h->st));
  return GPE_OK;
}

// Small fields: the CG's closing step applies the residual and cap tests from
// the update's partials itself (every one of its workgroups sums them), and
// the update needs no finalize launch.  Up to 256 partials (2^18 points) each
// thread of a workgroup loads at most one of them, so the sum costs the same
// there whatever the grid, however many workgroups repeat it.  A CG iteration
// with and without the finalize's launch, in c128 and c64: spin-3 256^2 141.8 ->
// 139.0 us, 135.2 -> 131.4;  512 x 384 244.5 -> 241.3, 185.2 -> 180.5;  64^3 271.0 -> 269.1,
// 213.1 -> 210.9;  spin-2 512^2 185.4 -> 182.0, 140.0 -> 139.0.
bool cg_local_step(const gpe_handle* h) { return h->nblk <= kRedThreads; }

template <typename T>
static gpe_status cg_step_t(gpe_handle* h, const void* p, const void* q, void* z, void* r) {
  CgArgs<T> a{p, q, z, r, h->part, 0.0, h->nel};
  a.adev = h->res + CG_ALPHA;
  a.skip = h->res + CG_DONE;
  GPE_KT(h, KK_VECTOR, launch_single(a, h->nblk, h->st));
  if (cg_local_step(h)) return GPE_OK;
  SlotCounts nb;
  for (int k = 0; k < kMaxQ; ++k) nb.nb[k] = h->nblk;
  GPE_KT(h, KK_FINALIZE, finalize(h->part, h->nblk, nb, 1, h->res, POST_CG_STEP, h->F, nullptr, h->ticket,
                                  h->res + CG_DONE, nullptr, h->st));
  return GPE_OK;
}

template <typename T>
static gpe_status cg_dir_t(gpe_handle* h, const void* r, void* p, void* z, int iter) {
  CgDirArgs<T> a{r, p, z, h->res, iter, h->nel};
  if (cg_local_step(h)) {
    a.part = h->part;
    a.nb = h->nblk;
  }
  GPE_KT(h, KK_VECTOR, launch_single(a, elementwise_blocks(h->nel), h->st));
  return GPE_OK;
}

gpe_status cg_dir_enq(gpe_handle* h, const void* r, void* p, void* z, int iter) {
  return work32(h) ? cg_dir_t<float>(h, r, p, z, iter) : cg_dir_t<double>(h, r, p, z, iter);
}

gpe_status cg_step_enq(gpe_handle* h, const void* p, const void* q, void* z, void* r) {
  return work32(h) ? cg_step_t<float>(h, p, q, z, r) : cg_step_t<double>(h, p, q, z, r);
}


gpe_status cg_state_read(gpe_handle* h, CgState* cs) {
  const double* c = h->hres;
  cs->done = c[CG_DONE] != 0.0;
  cs->reason = (int)c[CG_REASON];
  cs->iters = (int)c[CG_IT];
  cs->kappa = c[CG_KAPPA];
  cs->pp = c[CG_PP];
  if (cs->done && cs->reason == CG_STOP_CURVATURE) GPE_TRY(finite(h, c + CG_KAPPA, 2, "the CG curvature"));
  GPE_TRY(finite(h, c + CG_RR, 1, "the CG residual"));
  GPE_TRY(finite(h, c + CG_RR1, 1, "the CG residual"));
  return GPE_OK;
}

gpe_status prolong(const gpe_handle* c, const void* Xc, gpe_handle* f, void* Xf) {
  if (c->F != f->F || c->dim != f->dim) return fail(f, GPE_EINVAL, "prolong: problems differ");
  for (int a = 0; a < c->dim; ++a)
    if (f->n[a] != 2 * c->n[a]) return fail(f, GPE_EINVAL, "prolong: fine grid must have 2n points per axis");
  // ping-pong through the fine handle's scratch (T64, Gp); the set point is lost
  f->has_point = false;
  const void* src = Xc;
  size_t sizes[3] = {(size_t)c->n[0], (size_t)c->n[1], (size_t)c->n[2]};
  for (int a = 0; a < c->dim; ++a) {
    size_t inner = 1, outer = (size_t)c->K;
    for (int b = 0; b < a; ++b) inner *= sizes[b];
    for (int b = a + 1; b < c->dim; ++b) outer *= sizes[b];
    const bool last = a == c->dim - 1;
    void* dst = last ? Xf : (a == 0 ? f->T64 : f->Gp);
    const double scale = last ? std::pow(2.0, -0.5 * c->dim) : 1.0;
    GPE_HIP(f, prolong_axis(src, dst, c->ax[a].tw64, f->ax[a].tw64, c->n[a], inner, outer, scale, f->st));
    sizes[a] *= 2;
    src = dst;
  }
  GPE_HIP(f, hipStreamSynchronize(f->st));
  return GPE_OK;
}

}  // namespace gpe

using namespace gpe;

// ----------------------------------------------------------------- C ABI


// Validation of a problem statement (gpe_problem's contract); "" if valid.
static std::string problem_error(const gpe_problem* pr) {
  if (pr->F < 1 || pr->F > 3) return "F must be 1, 2 or 3";
  if (pr->dim < 1 || pr->dim > 3) return "dim must be 1, 2 or 3";
  if (!(std::fabs(pr->M) < pr->F)) return "|M| must be < F";
  if (pr->M < 0) return "M < 0: reverse the component order and pass -M";
  for (int a = 0; a < pr->dim; ++a) {
    const int n = pr->n[a];
    if (!lap_size_supported(n))
      return "n[" + std::to_string(a) + "] = " + std::to_string(n) + " unsupported (2^k or 3*2^k, 4..512)";
    if (!(pr->hi[a] > pr->lo[a])) return "empty box";
  }
  return "";
}

// ----------------------------------------------------------------- scratch of gpe_retract_noalloc
// The retraction's partial sums (3K slots of at most kMaxRedBlocks workgroups),
// the finalize's results and its ticket, for every admissible problem.  One
// copy per GPU, at a device address found once per device.
namespace {
constexpr size_t kNaPart = 3 * 7 * (size_t)kMaxRedBlocks;
constexpr size_t kNaRes = 64;
constexpr size_t kNaDoubles = kNaPart + kNaRes + 2;   // + the ticket (first 4 bytes of the last 16)
constexpr int kNaMaxDevices = 64;
}  // namespace
static __device__ __align__(256) double scratch[kNaDoubles];
static double* g_scratch_ptr[kNaMaxDevices];
static std::mutex g_scratch_mu;

// Device address of `scratch` on the current device (resolved once per device).
static gpe_status scratch_on_device(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(nullptr, e, "hipGetDevice");
  if (dev < 0 || dev >= kNaMaxDevices) return fail(nullptr, GPE_EINVAL, "device index beyond the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_fail(nullptr, e != hipSuccess ? e : hipErrorInvalidSymbol,
                                               "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return GPE_OK;
}

extern "C" {

const char* gpe_version(void) { return "gpe 0.1 (gfx950)"; }

void gpe_solve_opts_default(gpe_solve_opts* o) {
  if (!o) return;
  o->tol = 1e-6;
  o->maxit = 10000;
  o->retraction = GPE_R1_PROJECTIVE;
  o->rgbb_tol = 1e-2;
  o->rgbb_maxit = 2000;
  o->rgbb_rho = 1e-4;
  o->rgbb_delta = 0.2;
  o->rgbb_varrho = 0.85;
  o->rgbb_step0 = 0.1;
  o->eta1 = 0.01;
  o->eta2 = 0.9;
  o->gamma0 = 0.2;
  o->gamma1 = 1.0;
  o->gamma2 = 10.0;
  o->sigma_hat0 = 1.0;
  o->rho = 1e-4;
  o->delta = 0.2;
  o->alpha0 = 1.0;
  o->ls_max = 30;
  o->cg_maxit = 500;
  o->cg_T = 0.1;
  o->cg_theta = 1.0;
  o->max_reject_streak = 30;
  o->sigma_hat_min = 1e-8;
  o->verbose = 0;
  o->time_limit = 0.0;
  o->mg_levels = 0;
  o->mg_coarse_tol = 1e-5;
  o->polish_tol = 0.0;
  o->polish_window = 0;
  o->cg_per_digit = 80.0;
  o->trace = nullptr;
  o->trace_cap = 0;
}

const char* gpe_last_error(const gpe_handle* h) { return h ? h->err.c_str() : g_create_error.c_str(); }

gpe_status gpe_destroy(gpe_handle* h) {
  if (!h) return GPE_OK;
  (void)hipSetDevice(h->device);
  if (h->st) (void)hipStreamSynchronize(h->st);
  if (!h->res_shared) {
    if (h->res) (void)hipFree(h->res);
    if (h->hres) (void)hipHostFree(h->hres);
  }
  void* bufs[] = {h->ticket, h->V64, h->V32, h->part, h->gram_pt, h->gram_tmp, h->T64, h->T32, h->Xp, h->Gp, h->Xp32,
                  h->LX64, h->LX32,
                  h->tw[0], h->tw[1], h->tw[2], h->tw[3], h->tw[4], h->tw[5]};
  for (void* b : bufs)
    if (b) (void)hipFree(b);
  for (void* b : h->solver_bufs)
    if (b) (void)hipFree(b);
  for (auto& r : h->recs) {
    (void)hipEventDestroy(r.a);
    (void)hipEventDestroy(r.b);
  }
  for (auto e : h->event_pool) (void)hipEventDestroy(e);
  delete h;
  return GPE_OK;
}

gpe_status gpe_create(const gpe_problem* pr, const double* V, int precision, void* stream, gpe_handle** out) {
  if (!out) return fail(nullptr, GPE_EINVAL, "out is NULL");
  *out = nullptr;
  if (!pr || !V) return fail(nullptr, GPE_EINVAL, "problem or potential is NULL");
  if (precision != GPE_FP64 && precision != GPE_MIXED) return fail(nullptr, GPE_EINVAL, "bad precision");
  {
    const std::string err = problem_error(pr);
    if (!err.empty()) return fail(nullptr, GPE_EINVAL, err);
  }
  gpe_handle* h = new gpe_handle();
  h->prob = *pr;
  h->F = pr->F;
  h->K = 2 * pr->F + 1;
  h->dim = pr->dim;
  h->prec = precision;
  h->st = reinterpret_cast<hipStream_t>(stream);
  h->p = pr->p;
  h->q = pr->q;
  h->M = pr->M;
  for (int k = 0; k < 4; ++k) h->beta[k] = pr->beta[k];
  if (h->F < 3) h->beta[3] = 0;
  if (h->F < 2) h->beta[2] = 0;
  h->npts = 1;
  h->h = 1.0;
  for (int a = 0; a < h->dim; ++a) {
    h->n[a] = pr->n[a];
    h->lo[a] = pr->lo[a];
    h->hi[a] = pr->hi[a];
    h->npts *= (size_t)pr->n[a];
    h->h *= (pr->hi[a] - pr->lo[a]) / pr->n[a];
  }
  h->nel = h->npts * h->K;
  (void)hipGetDevice(&h->device);
  {
    // V may live in host or device memory: a device (or managed) pointer is
    // copied to the host mirror first; anything else is read as host memory
    hipPointerAttribute_t attr;
    bool on_device = false;
    if (hipPointerGetAttributes(&attr, V) == hipSuccess)
      on_device = attr.type == hipMemoryTypeDevice || attr.type == hipMemoryTypeManaged;
    else
      (void)hipGetLastError();
    h->Vhost.resize(h->npts);
    if (on_device) {
      const hipError_t ev = hipMemcpy(h->Vhost.data(), V, h->npts * sizeof(double), hipMemcpyDeviceToHost);
      if (ev != hipSuccess) {
        hip_fail(h, ev, "copy of the device potential");
        g_create_error = h->err;
        delete h;
        return GPE_EHIP;
      }
    } else {
      std::memcpy(h->Vhost.data(), V, h->npts * sizeof(double));
    }
  }
  const double* V_host = h->Vhost.data();

  // pointwise constants
  for (int i = 0; i < 7; ++i) {
    const double l = h->F - i;
    h->pw.zee[i] = i < h->K ? -h->p * l + h->q * l * l : 0.0;
    h->pw.zc[i] = 0.0;
  }
  for (int k = 0; k < 4; ++k) {
    h->pw.g[k] = 2.0 * h->beta[k] / h->h;
    h->pw.e[k] = h->beta[k] / (2.0 * h->h);
  }
  h->nblk = red_blocks(h->npts);

  gpe_status s;
#define GPE_ALLOC(ptr, bytes)                                              \
  do {                                                                     \
    s = alloc_field(h, (void**)&(ptr), (bytes));                           \
    if (s != GPE_OK) { g_create_error = h->err; gpe_destroy(h); return s; } \
  } while (0)
  const size_t f64 = h->nel * 16, f32 = h->nel * 8;
  GPE_ALLOC(h->V64, h->npts * sizeof(double));
  {
    size_t ps = kMaxRedBlocks;
    size_t inner = 1;
    for (int a = 0; a < h->dim; ++a) {
      LapAxis ax;
      ax.n = pr->n[a];
      ax.inner = (int)inner;
      ax.nlines = (long)(h->nel / pr->n[a]);
      const size_t m = lap_max_blocks(ax, h->K);
      if (m > ps) ps = m;
      inner *= (size_t)pr->n[a];
    }
    h->pstride = ps;
  }
  GPE_ALLOC(h->part, sizeof(double) * kMaxQ * h->pstride);
  GPE_ALLOC(h->res, sizeof(double) * kResDoubles);
  GPE_ALLOC(h->gram_pt, sizeof(double) * 8);
  GPE_ALLOC(h->gram_tmp, sizeof(double) * 8);
  GPE_ALLOC(h->ticket, sizeof(unsigned int) * 4);
  GPE_ALLOC(h->T64, f64);
  GPE_ALLOC(h->Xp, f64);
  GPE_ALLOC(h->Gp, f64);
  if (precision == GPE_FP64) GPE_ALLOC(h->LX64, f64);
  if (precision == GPE_MIXED) {
    GPE_ALLOC(h->LX32, f32);
    GPE_ALLOC(h->V32, h->npts * sizeof(float));
    GPE_ALLOC(h->T32, f32);
    GPE_ALLOC(h->Xp32, f32);
  }
  if (hipHostMalloc((void**)&h->hres, sizeof(double) * kResDoubles, hipHostMallocDefault) != hipSuccess) {
    g_create_error = "pinned host allocation failed";
    gpe_destroy(h);
    return GPE_ENOMEM;
  }
  auto bail = [&](hipError_t e, const char* w) {
    hip_fail(h, e, w);
    g_create_error = h->err;
    gpe_destroy(h);
    return GPE_EHIP;
  };
  hipError_t e = hipMemsetAsync(h->ticket, 0, sizeof(unsigned int) * 4, h->st);
  if (e != hipSuccess) return bail(e, "clear ticket");
  e = hipMemcpyAsync(h->V64, V_host, h->npts * sizeof(double), hipMemcpyHostToDevice, h->st);
  if (e != hipSuccess) return bail(e, "copy V");
  if (precision == GPE_MIXED) {
    std::vector<float> v32(h->npts);
    for (size_t j = 0; j < h->npts; ++j) v32[j] = (float)V_host[j];
    e = hipMemcpyAsync(h->V32, v32.data(), h->npts * sizeof(float), hipMemcpyHostToDevice, h->st);
    if (e != hipSuccess) return bail(e, "copy V32");
    e = hipStreamSynchronize(h->st);
    if (e != hipSuccess) return bail(e, "sync");
  }
  // Laplacian axes: axis a has lines of length n[a] at stride prod_{b<a} n[b]
  size_t inner = 1;
  for (int a = 0; a < h->dim; ++a) {
    const int n = h->n[a];
    LapAxis& ax = h->ax[a];
    ax.n = n;
    ax.inner = (int)inner;
    ax.nlines = (long)(h->nel / n);
    ax.lamc = 2.0 * M_PI / (h->hi[a] - h->lo[a]);
    std::vector<double> t64(2 * n);
    std::vector<float> t32(2 * n);
    for (int m = 0; m < n; ++m) {
      // exp(-2 pi i m / n), argument reduced exactly through m/n
      const double ang = -2.0 * M_PI * (double)m / (double)n;
      t64[2 * m] = std::cos(ang);
      t64[2 * m + 1] = std::sin(ang);
      t32[2 * m] = (float)t64[2 * m];
      t32[2 * m + 1] = (float)t64[2 * m + 1];
    }
    GPE_ALLOC(h->tw[2 * a], n * 16);
    GPE_ALLOC(h->tw[2 * a + 1], n * 8);
    e = hipMemcpy(h->tw[2 * a], t64.data(), n * 16, hipMemcpyHostToDevice);
    if (e != hipSuccess) return bail(e, "copy twiddles");
    e = hipMemcpy(h->tw[2 * a + 1], t32.data(), n * 8, hipMemcpyHostToDevice);
    if (e != hipSuccess) return bail(e, "copy twiddles");
    ax.tw64 = h->tw[2 * a];
    ax.tw32 = h->tw[2 * a + 1];
    inner *= (size_t)n;
  }
#undef GPE_ALLOC
  e = hipStreamSynchronize(h->st);
  if (e != hipSuccess) return bail(e, "sync");
  if (tune_xpass(h) != GPE_OK) {
    g_create_error = h->err;
    gpe_destroy(h);
    return GPE_EHIP;
  }
  *out = h;
  return GPE_OK;
}

gpe_status gpe_energy(gpe_handle* h, const void* X, double* E) {
  if (!h || !X || !E) return fail(h, GPE_EINVAL, "NULL argument");
  GPE_TRY(eval_enq(h, X, nullptr, nullptr));
  GPE_TRY(fetch(h));
  return eval_read(h, false, E, nullptr, nullptr);
}

gpe_status gpe_grad(gpe_handle* h, const void* X, void* G, int riemannian, double* E, double* gnorm) {
  if (!h || !X || !G) return fail(h, GPE_EINVAL, "NULL argument");
  if (X == G) return fail(h, GPE_EINVAL, "X and G must be distinct");
  double e, ag, bg;
  GPE_TRY(grad_enq(h, X, G, h->gram_tmp, riemannian ? GRAD_RIEM : GRAD_EUCLID, gnorm != nullptr));
  GPE_TRY(fetch(h));
  GPE_TRY(eval_read(h, true, &e, &ag, &bg));
  if (E) *E = e;
  if (riemannian || gnorm) {   // (formed for every Riemannian gradient, and checked with or without a taker)
    GPE_TRY(finite(h, h->hres + kResNorm, 1, "the gradient norm"));
    if (gnorm) *gnorm = std::sqrt(h->hres[kResNorm]);
  }
  return GPE_OK;
}

gpe_status gpe_set_point(gpe_handle* h, const void* X) {
  if (!h || !X) return fail(h, GPE_EINVAL, "NULL argument");
  // the kernels replace X_p, its Gram system and L X_p before the point can be
  // rejected: until it is accepted there is none
  h->has_point = false;
  // the multipliers and L X_p, which the HVP needs for <X_i, (LZ)_i> = <(LX)_i, Z_i>
  GPE_TRY(grad_enq(h, X, h->prec == GPE_MIXED ? h->T64 : h->LX64, h->gram_pt, GRAD_POINT, false));
  GPE_TRY(fetch(h));
  GPE_TRY(eval_read(h, true, &h->E_pt, &h->alpha_g, &h->beta_g));
  if (h->prec == GPE_MIXED && h->dim == 1) GPE_HIP(h, to_c64(h->T64, h->LX32, h->nel, h->st));
  h->has_point = true;
  return GPE_OK;
}

gpe_status gpe_hvp(gpe_handle* h, const void* Z, void* HZ, int riemannian, double sigma) {
  if (!h || !Z || !HZ) return fail(h, GPE_EINVAL, "NULL argument");
  if (Z == HZ) return fail(h, GPE_EINVAL, "Z and HZ must be distinct");
  return hvp(h, Z, HZ, riemannian != 0, sigma, nullptr, nullptr);
}

gpe_status gpe_hvp_dot(gpe_handle* h, const void* Z, void* HZ, double sigma, double* kappa) {
  if (!h || !Z || !HZ || !kappa) return fail(h, GPE_EINVAL, "NULL argument");
  if (Z == HZ) return fail(h, GPE_EINVAL, "Z and HZ must be distinct");
  return hvp(h, Z, HZ, true, sigma, kappa, nullptr);
}

gpe_status gpe_retract(gpe_handle* h, const void* X, const void* Xi, double t, int kind, void* Xout) {
  if (!h || !X || !Xout) return fail(h, GPE_EINVAL, "NULL argument");
  RetractNorms rn;
  GPE_TRY(retract_norms(h, X, Xi, false, &rn));
  GPE_TRY(retract_apply(h, rn, X, Xi, false, Xi ? t : 0.0, kind, Xout));
  GPE_HIP(h, hipStreamSynchronize(h->st));
  return GPE_OK;
}

gpe_status gpe_constraints(gpe_handle* h, const void* X, double* mass, double* mag) {
  if (!h || !X) return fail(h, GPE_EINVAL, "NULL argument");
  RetractNorms rn;
  GPE_TRY(retract_norms(h, X, nullptr, false, &rn));
  double m = 0, g = 0;
  for (int i = 0; i < h->K; ++i) {
    m += rn.uu[i];
    g += (h->F - i) * rn.uu[i];
  }
  if (mass) *mass = m;
  if (mag) *mag = g;
  return GPE_OK;
}

gpe_status gpe_project(gpe_handle* h, const void* X, const void* W, void* out) {
  if (!h || !X || !W || !out) return fail(h, GPE_EINVAL, "NULL argument");
  RetractNorms rn;
  GPE_TRY(retract_norms(h, X, W, false, &rn));
  double alpha, beta;
  GPE_TRY(proj_coeffs(h, rn, &alpha, &beta));
  double gn;
  GPE_TRY(project_grad(h, X, W, out, alpha, beta, &gn));
  return GPE_OK;
}

gpe_status gpe_prolong(const gpe_handle* coarse, const void* Xc, gpe_handle* fine, void* Xf) {
  if (!coarse || !fine || !Xc || !Xf) return fail(fine, GPE_EINVAL, "NULL argument");
  return gpe::prolong(coarse, Xc, fine, Xf);
}

gpe_status gpe_schedule(const gpe_handle* h, int* xpass_variant, float* variant_us, int nvariants) {
  if (!h) return fail(nullptr, GPE_EINVAL, "NULL handle");
  if (xpass_variant) *xpass_variant = h->xvar;
  for (int v = 0; v < nvariants && v < 3; ++v)
    if (variant_us) variant_us[v] = h->xvar_us[v];
  return GPE_OK;
}

gpe_status gpe_set_schedule(gpe_handle* h, int xpass_variant) {
  if (!h) return fail(nullptr, GPE_EINVAL, "NULL handle");
  const int nv = xpass_variants(h->n[0]);
  if (xpass_variant < 0 || xpass_variant >= nv)
    return fail(h, GPE_EINVAL, "x-pass variant " + std::to_string(xpass_variant) + " out of range: this grid has " +
                                   std::to_string(nv));
  h->xvar = xpass_variant;
  return GPE_OK;
}

gpe_status gpe_schedule_count(const gpe_handle* h, int* nvariants) {
  if (!h || !nvariants) return fail(nullptr, GPE_EINVAL, "NULL argument");
  *nvariants = xpass_variants(h->n[0]);
  return GPE_OK;
}

gpe_status gpe_timing_enable(gpe_handle* h, int enable) {
  if (!h) return fail(h, GPE_EINVAL, "NULL handle");
  GPE_HIP(h, hipStreamSynchronize(h->st));
  for (auto& r : h->recs) {
    h->event_pool.push_back(r.a);
    h->event_pool.push_back(r.b);
  }
  h->recs.clear();
  h->timing = enable != 0;
  return GPE_OK;
}

gpe_status gpe_timing_read(gpe_handle* h, int max, const char** names, int* counts, double* ms, int* nkinds) {
  if (!h) return fail(h, GPE_EINVAL, "NULL handle");
  GPE_HIP(h, hipStreamSynchronize(h->st));
  double tot[KK_COUNT] = {0};
  int cnt[KK_COUNT] = {0};
  for (auto& r : h->recs) {
    float t = 0.f;
    GPE_HIP(h, hipEventElapsedTime(&t, r.a, r.b));
    tot[r.kind] += t;
    cnt[r.kind] += 1;
  }
  int k = 0;
  for (int i = 0; i < KK_COUNT; ++i) {
    if (!cnt[i]) continue;
    if (k < max) {
      if (names) names[k] = kKernelNames[i];
      if (counts) counts[k] = cnt[i];
      if (ms) ms[k] = tot[i];
    }
    ++k;
  }
  if (nkinds) *nkinds = k;
  return GPE_OK;
}

gpe_status gpe_retract_noalloc(const gpe_problem* pr, const void* X, const void* Xi, double t, int kind, void* Xout,
                               void* stream) {
  if (!pr || !X || !Xout) return fail(nullptr, GPE_EINVAL, "NULL argument");
  {
    const std::string err = problem_error(pr);
    if (!err.empty()) return fail(nullptr, GPE_EINVAL, err);
  }
  if (kind != GPE_R1_PROJECTIVE && kind != GPE_R2_ORTHOGONAL && kind != GPE_R3_CLOSED)
    return fail(nullptr, GPE_EINVAL, "unknown retraction kind");
  const int F = pr->F, K = 2 * F + 1;
  size_t npts = 1;
  for (int a = 0; a < pr->dim; ++a) npts *= (size_t)pr->n[a];
  const int nblk = comp_blocks(npts);   // per component
  const int nq = Xi ? 3 * K : K;
  if ((size_t)3 * K * (size_t)nblk > kNaPart) return fail(nullptr, GPE_EINVAL, "problem exceeds the static scratch");
  double* base = nullptr;
  GPE_TRY(scratch_on_device(&base));
  double* part = base;
  double* res = base + kNaPart;
  unsigned int* ticket = reinterpret_cast<unsigned int*>(base + kNaPart + kNaRes);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
#define NA_HIP(call)                                                  \
  do {                                                                \
    hipError_t e_ = (call);                                           \
    if (e_ != hipSuccess) return hip_fail(nullptr, e_, #call);        \
  } while (0)
  // the ticket starts at 0 (a finalize leaves it there; an interrupted call might not)
  NA_HIP(hipMemsetAsync(ticket, 0, sizeof(unsigned int), st));
  NA_HIP((comp_norms<double, double>(K, X, Xi, part, nblk, npts, st)));
  SlotCounts nb;
  for (int q = 0; q < kMaxQ; ++q) nb.nb[q] = nblk;
  NA_HIP(finalize(part, nblk, nb, nq, res, POST_NONE, F, nullptr, ticket, nullptr, nullptr, st));
  double r[3 * 7];
  NA_HIP(hipMemcpyAsync(r, res, sizeof(double) * nq, hipMemcpyDeviceToHost, st));
  NA_HIP(hipStreamSynchronize(st));
  for (int i = 0; i < nq; ++i)
    if (!std::isfinite(r[i])) return fail(nullptr, GPE_ENUMERIC, "NaN or Inf in the component norms");
  double a[7], sig[7];
  for (int i = 0; i < K; ++i) {
    const double ux = Xi ? r[K + i] : 0.0, xx = Xi ? r[2 * K + i] : 0.0;
    a[i] = r[i] + 2.0 * t * ux + t * t * xx;   // ||u_i + t xi_i||^2
    if (a[i] < 0) a[i] = 0;
  }
  const int rs = kind == GPE_R1_PROJECTIVE ? sigma_projective(F, pr->M, a, sig)
               : kind == GPE_R2_ORTHOGONAL ? sigma_orthogonal(F, pr->M, a, sig)
                                           : sigma_closed(F, pr->M, a, sig);
  if (rs != SIGMA_OK)
    return fail(nullptr, GPE_EDOMAIN, kind == GPE_R3_CLOSED ? "retraction argument outside S"
                                                            : "retraction argument outside Omega");
  NA_HIP((scale_comps<double, double, double>(K, X, Xi, t, sig, Xout, npts, st)));
#undef NA_HIP
  return GPE_OK;
}

gpe_status gpe_newton_solve(gpe_handle* h, void* X, const gpe_solve_opts* opts, gpe_solve_stats* stats) {
  if (!h || !X) return fail(h, GPE_EINVAL, "NULL argument");
  gpe_solve_opts o;
  if (opts) o = *opts;
  else gpe_solve_opts_default(&o);
  gpe_solve_stats s;
  std::memset(&s, 0, sizeof(s));
  gpe_status r = newton_solve(h, X, &o, &s);
  if (stats) *stats = s;
  return r;
}

}  // extern "C"
