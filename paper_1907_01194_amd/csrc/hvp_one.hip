// The Hessian-vector product of a 1D grid (at most 512 points of each component)
// in one launch of one workgroup.  As an x pass, a finalize for the projection
// coefficients, a projection and (where kappa is wanted) a second finalize it
// is three or four launches of 2 to 8 us that depend on one another.  Bound by
// the launch and one thread's chain of operations.  Measured, spin-1 n = 128,
// c128, calls back to back: 14.0 -> 7.4 us (6.8 on the device).
#include "fft.h"

namespace gpe {

template <typename T, int N, int F>
__global__ void __launch_bounds__((XGeo<N, 2 * F + 1, XVAR_LATENCY>::THREADS))
hvp_one_kernel(const c_t<T>* __restrict__ X, const c_t<T>* __restrict__ Z, const c_t<T>* __restrict__ Y,
               const T* __restrict__ V, c_t<T>* __restrict__ W, const c_t<T>* __restrict__ twg, T lamc, PwParams p,
               const double* skip, OneArgs one) {
  xpass_body<T, N, F, XVAR_LATENCY, true>(X, Z, Y, V, W, twg, 1, (size_t)N, lamc, p, nullptr, 0, 0, skip, one);
}

template <typename T, int N, int F>
static hipError_t launch(const LapAxis& ax, const void* X, const void* Z, const void* Y, const T* V, void* W,
                   const PwParams& p, double* gram, double* res, double* mirror, int post, bool proj,
                   const double* skip, hipStream_t st) {
  using T2 = c_t<T>;
  using G = XGeo<N, 2 * F + 1, XVAR_LATENCY>;
  const size_t lds = sizeof(T2) * G::template lds_elems<T>();
  const hipError_t e = allow_lds(&hvp_one_kernel<T, N, F>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((hvp_one_kernel<T, N, F>), dim3(1), dim3(G::THREADS), lds, st, reinterpret_cast<const T2*>(X),
                     reinterpret_cast<const T2*>(Z), reinterpret_cast<const T2*>(Y), V, reinterpret_cast<T2*>(W),
                     reinterpret_cast<const T2*>(sizeof(T) == 8 ? ax.tw64 : ax.tw32), (T)ax.lamc, p, skip,
                     OneArgs{gram, res, mirror, post, proj});
  return hipGetLastError();
}

template <typename T>
hipError_t hvp_one(int F, const LapAxis& ax, const void* X, const void* Z, const void* Y, const T* V, void* W,
                   const PwParams& p, double* gram, double* res, double* mirror, int post, bool proj,
                   const double* skip, hipStream_t st) {
  switch (ax.n * 4 + F) {
#define GPE_CASE(NN)                                                                                                   \
  case NN * 4 + 1: return launch<T, NN, 1>(ax, X, Z, Y, V, W, p, gram, res, mirror, post, proj, skip, st); \
  case NN * 4 + 2: return launch<T, NN, 2>(ax, X, Z, Y, V, W, p, gram, res, mirror, post, proj, skip, st); \
  case NN * 4 + 3: return launch<T, NN, 3>(ax, X, Z, Y, V, W, p, gram, res, mirror, post, proj, skip, st);
    GPE_SIZES(GPE_CASE)
#undef GPE_CASE
    default: return hipErrorInvalidValue;
  }
}
template hipError_t hvp_one<double>(int, const LapAxis&, const void*, const void*, const void*, const double*, void*,
                                    const PwParams&, double*, double*, double*, int, bool, const double*, hipStream_t);
template hipError_t hvp_one<float>(int, const LapAxis&, const void*, const void*, const void*, const float*, void*,
                                   const PwParams&, double*, double*, double*, int, bool, const double*, hipStream_t);

}  // namespace gpe
