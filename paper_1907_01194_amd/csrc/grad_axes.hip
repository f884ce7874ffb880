// Strided axis passes of the energy and the gradient (FP64): the Parseval sum
// alone, or the accumulating pass with the projection, ||out||^2 and a c64
// result (see LapMode).
#include "fft.h"

namespace gpe {

template <int N, int MODE>
__global__ void __launch_bounds__((AxGeo<double, N, false>::THREADS))
grad_axis_kernel(const double2* __restrict__ in, const double2* acc, double2* out, float2* out32,
                 const double2* __restrict__ twg, int inner, double lamc, int F, size_t npts,
                 const double2* __restrict__ X, const double* __restrict__ coef, double* __restrict__ part,
                 size_t stride, int slot) {
  lap_body<double, N, false, 1, MODE>(in, acc, out, twg, inner, lamc, F, npts, X, coef, part, stride, slot,
                                      (long)blockIdx.x, nullptr, AbSrc{}, out32);
}

template <int N, int MODE>
static void launch(const LapAxis& ax, const void* in, const void* acc, void* out, void* out32, int F, size_t npts,
                   const void* X, const double* coef, double* part, size_t stride, int slot, int* tpc,
                   hipStream_t st) {
  using G = AxGeo<double, N, false>;
  const int grid = (int)ax_tiles<double, N, false>(2 * F + 1, npts);
  const size_t lds = sizeof(double2) * (size_t)(padded_len<double>(N) + G::TILE);
  hipLaunchKernelGGL((grad_axis_kernel<N, MODE>), dim3(grid), dim3(G::THREADS), lds, st,
                     reinterpret_cast<const double2*>(in), reinterpret_cast<const double2*>(acc),
                     reinterpret_cast<double2*>(out), reinterpret_cast<float2*>(out32),
                     reinterpret_cast<const double2*>(ax.tw64), ax.inner, ax.lamc, F, npts,
                     reinterpret_cast<const double2*>(X), coef, part, stride, slot);
  *tpc = grid / (2 * F + 1);
}

hipError_t grad_axis(const LapAxis& ax, bool sum_only, const void* in, const void* acc, void* out, void* out32, int F,
                     size_t npts, const void* X, const double* coef, double* part, size_t stride, int slot, int* tpc,
                     hipStream_t st) {
  switch (ax.n) {
#define GPE_CASE(NN)                                                                                                 \
  case NN:                                                                                                           \
    if (sum_only)                                                                                                    \
      launch<NN, LAP_SUM>(ax, in, nullptr, nullptr, nullptr, F, npts, nullptr, nullptr, part, stride, slot, tpc, st); \
    else                                                                                                             \
      launch<NN, LAP_FULL>(ax, in, acc, out, out32, F, npts, X, coef, part, stride, slot, tpc, st);                  \
    break;
    GPE_SIZES(GPE_CASE)
#undef GPE_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace gpe
