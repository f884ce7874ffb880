// Mesh transfer for the cascadic multigrid of Algorithm 1 (Sec. 5): the
// coarse mesh halves every axis of the same box (coarse node j = fine node
// 2j).  Prolongation is the Fourier (trigonometric) interpolant of the coarse
// samples, axis by axis; restriction is injection.  Both act on c128 fields of
// K components.
#include "fft.h"

namespace gpe {

// Samples half a mesh width further: times exp(i pi p / n) / n.  The Nyquist
// coefficient, split evenly between +-n/2, gives cos(pi n / 2 (2 j + 1) / n) = 0
// at the odd nodes.  tw2: exp(-i pi m / n), the twiddles of the fine axis.
struct HalfShift {
  const double2* __restrict__ tw2;
  template <int N, bool INV> __device__ __forceinline__ void apply(double2* v, int j) const {
    using St = Stage<N, make_plan(N).S - 1>;
#pragma unroll
    for (int k = 0; k < St::R; ++k) {
      const int f = St::freq(j, k);
      const int p = f < N / 2 ? f : f - N;
      double2 w = tw2[p < 0 ? -p : p];   // exp(-i pi |p| / n)
      if (p > 0) w.y = -w.y;
      v[k] = 2 * f == N ? mk<double2>(0.0, 0.0) : cscale(cmul(v[k], w), 1.0 / N);
    }
  }
};

// Lines of N values at stride `inner` to lines of 2 N: the even values are the
// line's own, the odd ones its half-shifted interpolant (one forward and one
// inverse transform).  Reads the coarse line once and writes the fine one once,
// bound by that traffic; as a 2N x N matrix product per line (each output a dot
// product over the coarse line, read by every output's thread) the three passes
// of 64^3 -> 128^3, spin 3, took 655, 465 and 933 us; now 26, 27 and 64 (88, 176
// and 352 MB), and the whole call 6517 -> 143 us without the host-built matrices.
template <int N, bool CONTIG>
__global__ void __launch_bounds__((AxGeo<double, N, CONTIG>::THREADS))
prolong_axis_kernel(const double2* __restrict__ in, double2* __restrict__ out, const double2* __restrict__ twg,
                    const double2* __restrict__ tw2, unsigned inner, size_t nlines, double scale) {
  using G = AxGeo<double, N, CONTIG>;
  using St = Stage<N, 0>;
  constexpr int TPL = G::TPL, LPB = G::LPB;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double2* tw = reinterpret_cast<double2*>(smem_raw);
  double2* lds = tw + padded_len<double>(N);
  const int t = threadIdx.x;
  if constexpr (St::S > 1)
    for (int m = t; m < N; m += blockDim.x) tw[lpad<double>(m)] = twg[m];
  const int ln = CONTIG ? t / TPL : t % LPB;
  const size_t line = (size_t)blockIdx.x * LPB + ln;
  LineCtx lc;
  lc.tl = CONTIG ? t % TPL : t / LPB;
  lc.lbase = CONTIG ? ln * G::LSTR : ln;
  lc.valid = ln < LPB && lc.tl < TPL && line < nlines;
  const size_t o = CONTIG ? line : line / inner, i0 = CONTIG ? 0 : line % inner;
  const double2* src = in + o * N * inner + i0;
  double2* dst = out + o * 2 * N * inner + i0;
  LineRegs<double, N> v;
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    const int j = lc.tl + i * TPL;
    if (lc.valid && St::has(j)) {
#pragma unroll
      for (int a = 0; a < St::R; ++a) {
        v[i][a] = src[(size_t)(j + a * St::M) * inner];
      }
    }
  }
  // strided lines store their even values at once; contiguous ones beside the
  // odd ones (each lane then fills whole 32 B pairs: 40 -> 26 us for 64^3, spin 3)
  LineRegs<double, N> even;
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    const int j = lc.tl + i * TPL;
    if (lc.valid && St::has(j)) {
#pragma unroll
      for (int a = 0; a < St::R; ++a) {
        if constexpr (CONTIG) even[i][a] = cscale(v[i][a], scale);
        else dst[(size_t)(2 * (j + a * St::M)) * inner] = cscale(v[i][a], scale);
      }
    }
  }
  if constexpr (St::S > 1) __syncthreads();   // the twiddle table
  line_apply<double, N, CONTIG ? 0 : LPB, G::kWave, true>(v, lds, tw, lc, HalfShift{tw2});
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    const int j = lc.tl + i * TPL;
    if (lc.valid && St::has(j)) {
#pragma unroll
      for (int a = 0; a < St::R; ++a) {
        if constexpr (CONTIG) dst[2 * (j + a * St::M)] = even[i][a];
        dst[(size_t)(2 * (j + a * St::M) + 1) * inner] = cscale(v[i][a], scale);
      }
    }
  }
}

template <int N, bool CONTIG>
static hipError_t launch(const void* in, void* out, const void* tw, const void* tw2, size_t inner, size_t outer,
                         double scale, hipStream_t st) {
  using G = AxGeo<double, N, CONTIG>;
  const size_t nlines = inner * outer, grid = (nlines + G::LPB - 1) / G::LPB;
  if (grid < 1 || grid > 0x7fffffff) return hipErrorInvalidValue;
  const size_t lds = sizeof(double2) * (size_t)(padded_len<double>(N) + G::TILE);
  hipLaunchKernelGGL((prolong_axis_kernel<N, CONTIG>), dim3((unsigned)grid), dim3(G::THREADS), lds, st,
                     reinterpret_cast<const double2*>(in), reinterpret_cast<double2*>(out),
                     reinterpret_cast<const double2*>(tw), reinterpret_cast<const double2*>(tw2), (unsigned)inner,
                     nlines, scale);
  return hipGetLastError();
}

// coarse lengths: twice the length has to be admissible too
#define GPE_COARSE_SIZES(M) M(4) M(6) M(8) M(12) M(16) M(24) M(32) M(48) M(64) M(96) M(128) M(192) M(256)

hipError_t prolong_axis(const void* in, void* out, const void* tw, const void* tw2, int n, size_t inner, size_t outer,
                        double scale, hipStream_t st) {
  switch (n) {
#define GPE_CASE(NN)                                                                        \
  case NN:                                                                                  \
    return inner == 1 ? launch<NN, true>(in, out, tw, tw2, inner, outer, scale, st)         \
                      : launch<NN, false>(in, out, tw, tw2, inner, outer, scale, st);
    GPE_COARSE_SIZES(GPE_CASE)
#undef GPE_CASE
    default: return hipErrorInvalidValue;
  }
}

// coarse[c][z][y][x] = scale * fine[c][2z][2y][2x]; nc = coarse sizes (x, y, z), unused axes 1
__global__ void restrict_kernel(const double2* __restrict__ fine, double2* __restrict__ coarse, int K, int ncx,
                                int ncy, int ncz, int sy, int sz, double scale) {
  const size_t npc = (size_t)ncx * ncy * ncz;
  const size_t total = npc * K;
  const size_t npf = (size_t)(ncx * 2) * (ncy * sy) * (ncz * sz);
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(e / npc);
    size_t r = e % npc;
    const int x = (int)(r % ncx);
    r /= ncx;
    const int y = (int)(r % ncy);
    const int z = (int)(r / ncy);
    const size_t nfx = (size_t)ncx * 2, nfy = (size_t)ncy * sy;
    const size_t jf = ((size_t)(z * sz) * nfy + (size_t)(y * sy)) * nfx + (size_t)(2 * x);
    double2 v = fine[(size_t)c * npf + jf];
    v.x *= scale;
    v.y *= scale;
    coarse[e] = v;
  }
}

hipError_t restrict_inject(const void* fine, void* coarse, int K, int dim, const int* nc, double scale,
                           hipStream_t st) {
  const int ncx = nc[0], ncy = dim > 1 ? nc[1] : 1, ncz = dim > 2 ? nc[2] : 1;
  const size_t total = (size_t)K * ncx * ncy * ncz;
  size_t g = (total + 255) / 256;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(restrict_kernel, dim3((unsigned)g), dim3(256), 0, st, reinterpret_cast<const double2*>(fine),
                     reinterpret_cast<double2*>(coarse), K, ncx, ncy, ncz, dim > 1 ? 2 : 1, dim > 2 ? 2 : 1, scale);
  return hipGetLastError();
}

}  // namespace gpe
