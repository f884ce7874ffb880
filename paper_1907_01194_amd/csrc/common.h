// Shared device/host helpers of the HIP library: complex arithmetic on the
// interleaved (re, im) storage, wavefront reductions and launch constants.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

namespace gpe {

template <typename T> struct cplx;
template <> struct cplx<double> { using type = double2; };
template <> struct cplx<float> { using type = float2; };
template <typename T> using c_t = typename cplx<T>::type;

template <typename T2> __host__ __device__ inline T2 mk(decltype(T2::x) re, decltype(T2::x) im) {
  T2 r; r.x = re; r.y = im; return r;
}
template <typename T2> __device__ __forceinline__ T2 cadd(T2 a, T2 b) { return mk<T2>(a.x + b.x, a.y + b.y); }
template <typename T2> __device__ __forceinline__ T2 csub(T2 a, T2 b) { return mk<T2>(a.x - b.x, a.y - b.y); }
template <typename T2> __device__ __forceinline__ T2 cmul(T2 a, T2 b) {
  return mk<T2>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) * b
template <typename T2> __device__ __forceinline__ T2 cmulc(T2 a, T2 b) {
  return mk<T2>(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
template <typename T2> __device__ __forceinline__ T2 cconj(T2 a) { return mk<T2>(a.x, -a.y); }
template <typename T2, typename S> __device__ __forceinline__ T2 cscale(T2 a, S s) {
  return mk<T2>(a.x * s, a.y * s);
}
template <typename T2> __device__ __forceinline__ decltype(T2::x) cabs2(T2 a) { return a.x * a.x + a.y * a.y; }
// Re(a * conj(b))
template <typename T2> __device__ __forceinline__ decltype(T2::x) cdotr(T2 a, T2 b) { return a.x * b.x + a.y * b.y; }

// Loads/stores of one complex element, both precisions.
template <typename T2> __device__ __forceinline__ T2 ld(const T2* p) { return *p; }

constexpr int kWave = 64;          // CDNA wavefront width
constexpr int kRedThreads = 256;   // block size of reduction-producing kernels
constexpr int kMaxQ = 32;          // partial sums per reduction launch (max)
constexpr int kMaxRedBlocks = 2048;
constexpr int kXcds = 8;           // accelerator dies (XCDs), each with its own L2

// The hardware hands workgroup b of a launch to XCD b % kXcds.  Renumbered
// this way, consecutive numbers share an XCD and its L2: workgroups that read
// neighbouring parts of the same cache lines then find them there.  A
// bijection on [0, nb) for any nb; workgroup 0 keeps number 0.
__device__ __forceinline__ int xcd_local_block(int b, int nb) {
  const int x = b % kXcds, i = b / kXcds, q = nb / kXcds, rem = nb % kXcds;
  return x * q + (x < rem ? x : rem) + i;
}

// Whether an elementwise pass over a field of `bytes` that an earlier pass has
// just gone through takes the last element first: a large field's end is what
// the 256 MB cache still holds (retraction scaling at spin-3 128^3, 235 MB: 120 ->
// 115 us), while a field that fits the XCDs' L2 (32 MB together) is best met in
// the same order, since the same workgroup numbers, hence XCDs, then read back
// what they wrote (256^2 spin-2, 5 MB: 6.2 -> 4.0 us).
__host__ __device__ __forceinline__ bool read_backwards(size_t bytes) { return bytes > ((size_t)32 << 20); }

// Sum of a double over the wavefront (shuffle tree).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Sums of NQ doubles per lane over the wavefront, all at once: while a lane
// still carries several of them, a step hands half to the partner lane and takes
// the partner's share of the other half, so NQ sums cost about NQ + 6 exchanges
// instead of 6 NQ (7 sums: 10 instead of 42, 15 sums: 17 instead of 90).  With
// it the gradient's x pass (11 sums at spin 2) takes 10.4 us instead of 12.2 at
// 256^2 and 46 instead of 52 at 96^3, the batched x pass of 64 problems 49 not 53.  On
// return v[0] of lane l is the sum of quantity wave_slot<NQ>(l) (lanes whose slot
// is NQ or more hold nothing); the order of the additions is fixed.
template <int NQ> __host__ __device__ constexpr int pow2_ceil() {
  int p = 1;
  while (p < NQ) p *= 2;
  return p;
}
template <int NQ> __device__ __forceinline__ int wave_slot(int lane) {
  constexpr int P = pow2_ceil<NQ>();
  int q = 0;
  for (int w = P / 2, off = kWave / 2; w > 0; w >>= 1, off >>= 1) q += lane & off ? w : 0;
  return q;
}
template <int NQ> __device__ __forceinline__ void wave_sums(double (&v)[pow2_ceil<NQ>()], int lane) {
  constexpr int P = pow2_ceil<NQ>();
  static_assert(P <= kWave, "one quantity per lane at most");
  int off = kWave / 2;
#pragma unroll
  for (int w = P / 2; w > 0; w >>= 1, off >>= 1) {
    const bool up = lane & off;   // this lane keeps the upper half
#pragma unroll
    for (int q = 0; q < w; ++q) {
      const double lo = v[q], hi = v[q + w];
      v[q] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, off, kWave);
    }
  }
#pragma unroll
  for (; off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off, kWave);
}

// Block-reduce NQ per-thread doubles (any blockDim.x <= 1024, a multiple of the
// wave size): thread q calls sink(q, sum q) for q < NQ.  block_partials_any: the
// sums go to part[q * stride + blk].
template <int NQ, typename Sink>
__device__ inline void block_sums(const double (&acc)[NQ], Sink&& sink) {
  constexpr int P = pow2_ceil<NQ>();
  __shared__ double red[1024 / kWave][P];
  const int lane = threadIdx.x % kWave;
  const int wid = threadIdx.x / kWave;
  const int nw = (blockDim.x + kWave - 1) / kWave;
  double v[P];
#pragma unroll
  for (int q = 0; q < P; ++q) v[q] = q < NQ ? acc[q < NQ ? q : 0] : 0.0;
  wave_sums<NQ>(v, lane);
  if (lane % (kWave / P) == 0) red[wid][wave_slot<NQ>(lane)] = v[0];
  __syncthreads();
  if (threadIdx.x < NQ) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w][threadIdx.x];
    sink((int)threadIdx.x, s);
  }
}
template <int NQ>
__device__ inline void block_partials_any(const double (&acc)[NQ], double* __restrict__ part, size_t stride,
                                          size_t blk) {
  block_sums(acc, [&](int q, double s) { part[(size_t)q * stride + blk] = s; });
}

// Let a kernel take `lds` bytes of dynamic LDS (up to 64 KB need no asking).
template <typename Kernel> inline hipError_t allow_lds(Kernel* kernel, size_t lds) {
  if (lds <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lds);
}

// Workgroups of a reduction over npts grid points: four points per thread, but
// no fewer than one per thread up to 256 workgroups (a small field's reduction is
// bound by each thread's chain of loads: the CG update of a 256^2 spin-2 field
// takes 10.2 us with 64 workgroups and 5.7 with 256).
inline int red_blocks(size_t npts) {
  const size_t wide = (npts + kRedThreads - 1) / kRedThreads;
  size_t b = (npts + kRedThreads * 4 - 1) / (kRedThreads * 4);
  if (b < 256) b = wide < 256 ? wide : 256;
  if (b < 1) b = 1;
  if (b > (size_t)kMaxRedBlocks) b = kMaxRedBlocks;
  return (int)b;
}

// Workgroups per component of a reduction that keeps the components' sums
// apart: each takes one component's points, so it streams two or four arrays,
// not that many per component (K of them a power of two apart), and carries a
// few sums instead of several per component.
inline int comp_blocks(size_t npts) {
  size_t b = (npts + kRedThreads * 2 - 1) / (kRedThreads * 2);
  if (b < 1) b = 1;
  if (b > 512) b = 512;
  return (int)b;
}

}  // namespace gpe
