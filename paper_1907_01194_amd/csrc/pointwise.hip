// Pointwise energy density and gradient (Sec. 3) over a field whose Laplacian
// is at hand: the form the batched evaluations take (one launch for many
// problems).  A lone handle fuses these terms into its x-axis pass (grad_x.h).
#include "spin.h"
#include "batch_ops.h"

namespace gpe {

template <typename T, int F>
__device__ void run_op(const PwGradArgs<T, F>& a, int blk, int nblk) {
  using T2 = c_t<T>;
  auto X = reinterpret_cast<const T2*>(a.X);
  auto LX = reinterpret_cast<const T2*>(a.LX);
  auto V = reinterpret_cast<const T*>(a.V);
  auto G = reinterpret_cast<T2*>(a.G);
  const size_t n = a.npts;
  constexpr int K = 2 * F + 1;
  constexpr int NQ = 1 + 2 * K;
  double acc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
  for (size_t j = (size_t)blk * blockDim.x + threadIdx.x; j < n; j += (size_t)nblk * blockDim.x) {
    T2 x[K], lx[K];
    T kin = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      x[i] = X[i * n + j];
      lx[i] = LX[i * n + j];
      kin += T(0.5) * cdotr(lx[i], x[i]);
      acc[1 + K + i] += (double)cabs2(x[i]);
    }
    const T e = grad_point<T, F>(x, V[j], a.p, [&](int i, T2 qi) {
      const T2 g = cadd(lx[i], qi);
      G[i * n + j] = g;
      acc[1 + i] += (double)cdotr(x[i], g);
    });
    acc[0] += (double)kin + (double)e;
  }
  block_partials_any<NQ>(acc, a.part, nblk, blk);
}

GPE_OP(PwGradArgs<double, 1>)
GPE_OP(PwGradArgs<double, 2>)
GPE_OP(PwGradArgs<double, 3>)
}  // namespace gpe
