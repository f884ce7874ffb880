// Fused x pass of the energy and the gradient (Sec. 3), FP64: one read of X and
// V gives the pointwise energy density and gradient terms and L_x X of the same
// rows.  Included once per spin F (GPE_GRAD_F) so that the three compile side by
// side.
//
// With LX formed in full first, a gradient reads and writes 11 fields in 3D (x
// 2, y 3, z 3, pointwise 3) and an energy 10.  Here the x pass writes G = L_x X +
// q at once and the other axes accumulate into it (8 fields), and every kinetic
// sum <X_i, L_a X_i> comes from Parseval inside its pass, so an energy needs the
// forward transforms only and writes nothing (3 fields).  Bound by HBM on large
// grids (spin-2 96^3: 46 us for 2 fields and V with the gradient's sums, 22 us for
// the energy's one) and by latency on small ones (256^2: 12 us).  Measured, with
// the results stored in pinned memory by the finalize instead of a copy:
//   energy, spin-1 512^2 (4 launches -> 2) 56.5 -> 28.6 us;
//   Riemannian gradient, spin-2 256^2 (7 launches, 2 synchronisations -> 4, 1) 75.9 -> 39.9 us;
//   energy, gradient, set point and product, spin-2 96^3 (autograd) 984 -> 620 us.
#include "fft.h"

namespace gpe {

// GRAD: G = L_x X + q (point: G = L_x X alone), the partial sums
//   [0] pointwise energy + 1/2 <X, L_x X>, [1 + i] <X_i, q_i + (L_x X)_i>, [1 + K + i] ||X_i||^2,
// and copies of X to xc (c128) and xc32 (c64) where given.  !GRAD: [0] only.
// ONE (1D grids, one workgroup): the sums' post-operation, the projection and the
// norm of G follow in the same launch (a Riemannian gradient of spin-1 n = 128 with
// its host round trip 48.0 -> 21.9 us, an energy 25.0 -> 16.1, a set point 32 -> 18).
struct GradOne {
  double* gram = nullptr;
  double* res = nullptr;
  double* mirror = nullptr;
  bool proj = false, norm = false;
};

// SUMS: the workgroups from nbx on take the tiles of the strided axes' Parseval
// sums.  They read X alone, like the x pass, and a launch of their own waits for
// it for nothing: on small grids one latency instead of two or three (spin-1 48^3,
// energy 26.5 -> 20.8 us; 512^2 31.2 -> 28.6), on large ones their transforms fill
// the x pass' waits (spin-2 96^3, energy 69.9 -> 56.3, Riemannian gradient 151 ->
// 144).  Axes of the x axis' length only (one kernel per length, not per pair).
template <int N, int F, int VAR> constexpr int sums_threads() {
  constexpr int a = XGeo<N, 2 * F + 1, VAR>::THREADS, b = AxGeo<double, N, false>::THREADS;
  return a > b ? a : b;
}
template <int N, int F, bool GRAD, int VAR, bool ONE = false, bool SUMS = false>
__global__ void __launch_bounds__((SUMS ? sums_threads<N, F, VAR>() : XGeo<N, 2 * F + 1, VAR>::THREADS), 2)
grad_xpass_kernel(const double2* __restrict__ X, const double* __restrict__ V, double2* __restrict__ G,
                  double2* __restrict__ xc, float2* __restrict__ xc32, const double2* __restrict__ twg, long nrows,
                  size_t npts, double lamc, PwParams p, bool point, double* __restrict__ part, size_t stride,
                  GradOne one, SumAxes sums, int nbx) {
  if constexpr (SUMS) {
    if ((int)blockIdx.x >= nbx) {   // uniform over the workgroup
      const int tiles = (2 * F + 1) * sums.tpc, b = (int)blockIdx.x - nbx, k = b < tiles ? 0 : 1;
      lap_body<double, N, false, 1, LAP_SUM>(X, nullptr, nullptr, twg, sums.inner[k], sums.lamc[k], F, npts, nullptr,
                                             nullptr, part, stride, sums.slot[k], (long)(b - k * tiles), nullptr,
                                             AbSrc{});
      return;
    }
  }
  using T = double;
  using T2 = double2;
  constexpr int K = 2 * F + 1;
  using GG = XGeo<N, K, VAR>;
  using St = Stage<N, 0>;
  constexpr int TPL = GG::TPL, RPB = GG::RPB, LINES = GG::LINES, PPT = GG::PPT;
  constexpr int LSTR = GG::template lstr<T>();
  constexpr int NQ = GRAD ? 1 + 2 * K : 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T2* tw = reinterpret_cast<T2*>(smem_raw);
  T2* lds = tw + LSTR;
  const int t = threadIdx.x;
  if constexpr (St::S > 1)
    for (int m = t; m < N; m += blockDim.x) tw[lpad<T>(m)] = twg[m];
  double acc[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) acc[i] = 0.0;
  const long row0 = (long)blockIdx.x * RPB;
  const size_t r0 = (size_t)row0 * N;
  const unsigned np = SUMS && t >= GG::THREADS ? 0 : (unsigned)(nrows - row0 < RPB ? nrows - row0 : RPB) * N;

  // ---- pointwise terms of this thread's points; the rows of X go to LDS
  // Where a workgroup has several rows, all of a thread's points are fetched before
  // the first is used: LDS and registers hold the CU to 2-4 wavefronts per SIMD, too
  // few to cover one point's loads at a time.  256 x 256 x 64, gradient of spin 1, 2, 3:
  // 116 -> 106 us, 186 -> 179, 265 -> 251, although 256 points of spin 1, 2 and 3 spill 6,
  // 12 and 10 registers (spin 3 also point by point); spin-3 128^3 energy 128 -> 121.
  // Grids whose workgroups are few lose a little: 256 x 64 x 32 spin 2 30.5 -> 31.8 us.
  // One row a workgroup is faster point by point (512^2: 15.5 us against 16.6).
  constexpr bool AHEAD = RPB > 1;
  T2 xs[AHEAD ? PPT : 1][K], q[GRAD ? PPT : 1][K];
  T vs[AHEAD ? PPT : 1];
  auto fetch = [&](int pp, T2(&x)[K], T& vj) {
    const unsigned pt = t + pp * GG::THREADS;
    if (pt < np) {
#pragma unroll
      for (int i = 0; i < K; ++i) x[i] = at(X + r0 + i * npts, pt * (unsigned)sizeof(T2));
      vj = at(V + r0, pt * (unsigned)sizeof(T));
    }
  };
  if constexpr (AHEAD) {
#pragma unroll
    for (int pp = 0; pp < PPT; ++pp) fetch(pp, xs[pp], vs[pp]);
  }
#pragma unroll
  for (int pp = 0; pp < PPT; ++pp) {
    const unsigned pt = t + pp * GG::THREADS;
    if (pt < np) {
      const unsigned ob = pt * (unsigned)sizeof(T2);
      if constexpr (!AHEAD) fetch(pp, xs[0], vs[0]);
      const T2(&x)[K] = xs[AHEAD ? pp : 0];
      const T vj = vs[AHEAD ? pp : 0];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        lds[(i * RPB + pt / N) * LSTR + lpad<T>(pt % N)] = x[i];
        if constexpr (GRAD) acc[1 + K + i] += cabs2(x[i]);
      }
      acc[0] += grad_point<T, F>(x, vj, p, [&](int i, T2 qi) {
        if constexpr (GRAD) {
          acc[1 + i] += cdotr(x[i], qi);
          q[pp][i] = qi;
        }
      });
      if constexpr (GRAD) {
        if (xc)
#pragma unroll
          for (int i = 0; i < K; ++i) at(xc + r0 + i * npts, ob) = x[i];
        if (xc32)
#pragma unroll
          for (int i = 0; i < K; ++i)
            at(xc32 + r0 + i * npts, pt * (unsigned)sizeof(float2)) = mk<float2>((float)x[i].x, (float)x[i].y);
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // one point at a time
  }
  __syncthreads();

  // ---- L_x X of every component's rows, in place in LDS
  LineCtx lc;
  const int ls = t / TPL;
  lc.tl = t % TPL;
  lc.valid = ls < LINES && row0 + ls % RPB < nrows;
  lc.lbase = ls * LSTR;
  LineRegs<T, N> v;
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    const int j = lc.tl + i * TPL;
    if (lc.valid && St::has(j)) {
#pragma unroll
      for (int a = 0; a < St::R; ++a) v[i][a] = lds[lds_at<T, St::R, St::M, 0>(lc.lbase, j, a)];
    }
  }
  double pars = 0.0;
  line_apply<T, N, 0, GG::kWave, GRAD>(v, lds, tw, lc, LambdaScale<T>{lamc, T(1) / T(N), pars});
  acc[0] += 0.5 * pars;
  if constexpr (GRAD) {
#pragma unroll
    for (int i = 0; i < K; ++i) acc[1 + i] += ls / RPB == i ? pars : 0.0;
#pragma unroll
    for (int i = 0; i < St::NB; ++i) {
      const int j = lc.tl + i * TPL;
      if (lc.valid && St::has(j)) {
#pragma unroll
        for (int a = 0; a < St::R; ++a) lds[lds_at<T, St::R, St::M, 0>(lc.lbase, j, a)] = v[i][a];
      }
    }
    __syncthreads();
  }
  __shared__ double sum[ONE ? 16 : 1], state[ONE ? 64 : 1];
  if constexpr (ONE) {
    if (t < 64) state[t] = one.res[t];
    block_sums(acc, [&](int k, double s) { sum[k] = s; });
    __syncthreads();
    if (t == 0) finalize_post(sum, NQ, state, one.res, GRAD ? POST_GRAD : POST_ENERGY, F, one.gram, nullptr);
    __syncthreads();
  }
  double nrm[1] = {0.0};
  if constexpr (GRAD) {
#pragma unroll
    for (int pp = 0; pp < PPT; ++pp) {
      const unsigned pt = t + pp * GG::THREADS;
      if (pt < np) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const T2 l = lds[(i * RPB + pt / N) * LSTR + lpad<T>(pt % N)];
          T2 g = point ? l : cadd(l, q[pp][i]);
          if constexpr (ONE) {
            if (one.proj) {
              const double c = state[1 + 2 * K] + state[2 + 2 * K] * (double)(F - i);
              const T2 xv = at(X + r0 + i * npts, pt * (unsigned)sizeof(T2));
              g.x -= c * xv.x;
              g.y -= c * xv.y;
            }
            nrm[0] += cabs2(g);
          }
          at(G + r0 + i * npts, pt * (unsigned)sizeof(T2)) = g;
        }
      }
    }
  }
  if constexpr (ONE) {
    if (GRAD && one.norm) {
      block_sums(nrm, [&](int, double s) { one.res[kResNorm] = state[kResNorm] = s; });
      __syncthreads();
    }
    if (one.mirror && t < 64) one.mirror[t] = state[t];
  } else {
    block_partials_any<NQ>(acc, part, stride, blockIdx.x);
  }
}

template <int N, int F, int VAR, bool RIDE>
static hipError_t launch_gx(const LapAxis& ax, size_t npts, const void* X, const double* V, void* G, void* xc, void* xc32,
                      const PwParams& p, bool point, double* part, size_t stride, int* nb, SumAxes* sums, hipStream_t st) {
  using GG = XGeo<N, 2 * F + 1, VAR>;
  using AG = AxGeo<double, N, false>;
  const long nrows = (long)(npts / N);
  const int grid = (int)((nrows + GG::RPB - 1) / GG::RPB);
  const int tiles = RIDE ? (int)ax_tiles<double, N, false>(2 * F + 1, npts) : 0;
  sums->tpc = tiles / (2 * F + 1);
  size_t elems = GG::template lds_elems<double>();
  if (RIDE && elems < (size_t)padded_len<double>(N) + AG::TILE) elems = (size_t)padded_len<double>(N) + AG::TILE;
  const size_t lds = sizeof(double2) * elems;
  auto run = [&](auto* kernel) {
    const hipError_t e = allow_lds(kernel, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid + sums->n * tiles), dim3(RIDE ? sums_threads<N, F, VAR>() : GG::THREADS),
                       lds, st, reinterpret_cast<const double2*>(X), V,
                       reinterpret_cast<double2*>(G), reinterpret_cast<double2*>(xc), reinterpret_cast<float2*>(xc32),
                       reinterpret_cast<const double2*>(ax.tw64), nrows, npts, ax.lamc, p, point, part, stride,
                       GradOne{}, *sums, grid);
    return hipGetLastError();
  };
  *nb = grid;
  return G ? run(&grad_xpass_kernel<N, F, true, VAR, false, RIDE>) : run(&grad_xpass_kernel<N, F, false, VAR, false, RIDE>);
}

// From kLatencyPoints on 256 threads' rows a workgroup, against 128: gradient and
// energy of spin-2 96^3 46.7, 24.0 -> 46.4, 22.8 us, of spin-1 256 x 256 x 64 126.6,
// 58.5 -> 125.5, 51.7 (fewer partial sums, and one twiddle table for twice the rows).
// With other axes' sums in the launch 128, the threads of most of their tiles (the
// rest of a workgroup would idle): energy of spin-2 96^3 72.6 -> 56.3 us, of spin-3
// 128^3 172 -> 140 (in launches of their own 69.9 and 154.5).
template <int F>
hipError_t grad_xpass(const LapAxis& ax, size_t npts, const void* X, const double* V, void* G, void* xc, void* xc32,
                      const PwParams& p, bool point, double* part, size_t stride, int* nb, SumAxes* sums,
                      hipStream_t st) {
  switch (ax.n) {
#define GPE_GX(NN, VAR, RIDE) \
  return launch_gx<NN, F, VAR, RIDE>(ax, npts, X, V, G, xc, xc32, p, point, part, stride, nb, sums, st)
#define GPE_CASE(NN)                                               \
  case NN: {                                                       \
    constexpr bool mid = mid_length(NN);                           \
    const bool small = mid && npts < kLatencyPoints;               \
    if (small && sums->n) GPE_GX(NN, (mid ? XVAR_LATENCY : 1), true);   \
    if (small) GPE_GX(NN, (mid ? XVAR_LATENCY : 2), false);        \
    if (sums->n) GPE_GX(NN, 1, true);                              \
    GPE_GX(NN, 2, false);                                          \
  }
    GPE_SIZES(GPE_CASE)
#undef GPE_CASE
#undef GPE_GX
    default: return hipErrorInvalidValue;
  }
}
template <int N, int F>
static hipError_t launch_one(const LapAxis& ax, const void* X, const double* V, void* G, void* xc, void* xc32,
                       const PwParams& p, bool point, const GradOne& one, hipStream_t st) {
  using GG = XGeo<N, 2 * F + 1, XVAR_LATENCY>;
  const size_t lds = sizeof(double2) * GG::template lds_elems<double>();
  auto run = [&](auto* kernel) {
    const hipError_t e = allow_lds(kernel, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(GG::THREADS), lds, st, reinterpret_cast<const double2*>(X), V,
                       reinterpret_cast<double2*>(G), reinterpret_cast<double2*>(xc), reinterpret_cast<float2*>(xc32),
                       reinterpret_cast<const double2*>(ax.tw64), 1, (size_t)N, ax.lamc, p, point, nullptr, 0, one,
                       SumAxes{}, 1);
    return hipGetLastError();
  };
  return G ? run(&grad_xpass_kernel<N, F, true, XVAR_LATENCY, true>) : run(&grad_xpass_kernel<N, F, false, XVAR_LATENCY, true>);
}

template <int F>
hipError_t grad_one(const LapAxis& ax, const void* X, const double* V, void* G, void* xc, void* xc32,
                    const PwParams& p, bool point, bool proj, bool norm, double* gram, double* res, double* mirror,
                    hipStream_t st) {
  const GradOne one{gram, res, mirror, proj, norm};
  switch (ax.n) {
#define GPE_CASE(NN) \
  case NN: return launch_one<NN, F>(ax, X, V, G, xc, xc32, p, point, one, st);
    GPE_SIZES(GPE_CASE)
#undef GPE_CASE
    default: return hipErrorInvalidValue;
  }
}
template hipError_t grad_one<GPE_GRAD_F>(const LapAxis&, const void*, const double*, void*, void*, void*,
                                         const PwParams&, bool, bool, bool, double*, double*, double*, hipStream_t);
template hipError_t grad_xpass<GPE_GRAD_F>(const LapAxis&, size_t, const void*, const double*, void*, void*, void*,
                                           const PwParams&, bool, double*, size_t, int*, SumAxes*, hipStream_t);

}  // namespace gpe
