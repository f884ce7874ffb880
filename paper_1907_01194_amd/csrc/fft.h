// Device building blocks of the spectral Laplacian passes (Sec. 3, eq.
// discrete:laplace): line transforms with each thread holding a whole
// butterfly in registers, one axis pass over a tile of lines, and the fused x
// pass of the Hessian-vector product (pointwise Hessian terms of Sec. 3 plus
// L_x).  The bodies take their workgroup index explicitly so that one batched
// launch can run them for many problems (batch_fft.hip) as well as one
// (lap.hip).
//
// L_a of a line is DFT, multiply by lambda^2 / n, inverse DFT.  The forward
// transform is decimation in frequency in place (natural order in, digit-
// reversed out), the inverse its mirror image (digit-reversed in, natural
// out), so no reordering pass exists and:
//   * a stage reads and writes the same LDS elements from the same thread, so
//     only the hand-over between two stages needs a barrier;
//   * the last forward stage, the scaling and the first inverse stage act on
//     the same elements and stay in registers.
// A line of n = r0 r1 thus crosses LDS twice (once per direction), where a
// self-sorting transform of three radix <= 8 stages crosses it five times.
#pragma once

#include "common.h"
#include <type_traits>

#include "finalize.h"
#include "kernels.h"
#include "spin.h"

namespace gpe {

// Stages of a line and the threads that share it.  Two stages where the larger
// radix fits the registers (<= 16 complex values per thread), else three.  T
// divides the wavefront for every length except 384 (T = 48), so that the
// threads of one line sit in one wavefront wherever lines are contiguous.
struct RadixPlan {
  int S;
  int r[3];
  int T;
};

constexpr RadixPlan make_plan(int N) {
  switch (N) {
    case 4: return {1, {4, 1, 1}, 1};
    case 6: return {1, {6, 1, 1}, 1};
    case 8: return {1, {8, 1, 1}, 1};
    case 12: return {2, {3, 4, 1}, 4};
    case 16: return {2, {4, 4, 1}, 4};
    case 24: return {2, {6, 4, 1}, 4};
    case 32: return {2, {8, 4, 1}, 4};
    case 48: return {2, {6, 8, 1}, 8};
    case 64: return {2, {8, 8, 1}, 8};
    case 96: return {2, {12, 8, 1}, 8};
    case 128: return {2, {16, 8, 1}, 8};
    case 192: return {2, {12, 16, 1}, 16};
    case 256: return {2, {16, 16, 1}, 16};
    case 384: return {3, {8, 8, 6}, 48};
    case 512: return {3, {8, 8, 8}, 64};
    default: return {0, {1, 1, 1}, 1};
  }
}

constexpr int plan_prefix(RadixPlan p, int s) {
  int v = 1;
  for (int i = 0; i < s; ++i) v *= p.r[i];
  return v;
}

// Stage s of a line: N / R butterflies of R elements at stride M; butterfly j
// holds the elements base(j) + a M, a = 0..R-1; a thread takes the
// butterflies tl, tl + T, ... (NB of them).
template <int N, int s> struct Stage {
  static constexpr RadixPlan P = make_plan(N);
  static constexpr int S = P.S, T = P.T;
  static constexpr int R = P.r[s];
  static constexpr int M = N / plan_prefix(P, s + 1);
  static constexpr int NBF = N / R;
  static constexpr int NB = (NBF + T - 1) / T;
  static constexpr bool kFull = NBF % T == 0;
  static __host__ __device__ constexpr int base(int j) { return s == 0 ? j : (j / M) * (M * R) + j % M; }
  static __host__ __device__ constexpr bool has(int j) { return kFull || j < NBF; }
  // frequency of output k of butterfly j of the last stage (digits of the location reversed)
  static __host__ __device__ constexpr int freq(int j, int k) {
    return S == 1 ? k : S == 2 ? j + P.r[0] * k : j / P.r[1] + P.r[0] * (j % P.r[1]) + P.r[0] * P.r[1] * k;
  }
};

// multiply by -i (forward) or +i (inverse)
template <bool FWD, typename T2> __device__ __forceinline__ T2 mul_mi(T2 a) {
  return FWD ? mk<T2>(a.y, -a.x) : mk<T2>(-a.y, a.x);
}

// cos(2 pi m / 48); every radix up to 16 divides 48
__host__ __device__ constexpr double cos48(int m) {
  constexpr double c[13] = {1.0, 0.9914448613738104, 0.9659258262890683, 0.9238795325112867, 0.8660254037844387,
                            0.7933533402912352, 0.7071067811865476, 0.6087614290087207, 0.5, 0.38268343236508977,
                            0.25881904510252074, 0.13052619222005157, 0.0};
  m = ((m % 48) + 48) % 48;
  if (m > 24) m = 48 - m;
  return m <= 12 ? c[m] : -c[24 - m];
}

// a * exp(-+ 2 pi i M / R) with the factor known at compile time
template <int R, int M, bool FWD, typename T2> __device__ __forceinline__ T2 mul_w(T2 a) {
  using T = decltype(T2::x);
  static_assert(48 % R == 0, "constants are multiples of 2 pi / 48");
  constexpr int m = M % R;
  if constexpr (m == 0) return a;
  else if constexpr (4 * m == R) return mul_mi<FWD>(a);
  else if constexpr (2 * m == R) return mk<T2>(-a.x, -a.y);
  else {
    constexpr T c = (T)cos48(m * (48 / R));
    constexpr T s = (T)((FWD ? -1.0 : 1.0) * cos48(m * (48 / R) - 12));   // sin t = cos(t - pi/2)
    return mk<T2>(a.x * c - a.y * s, a.x * s + a.y * c);
  }
}

template <int R, bool FWD, typename T2> struct Dft;

template <bool FWD, typename T2> struct Dft<2, FWD, T2> {
  __device__ static __forceinline__ void run(T2* a) {
    T2 t = a[0];
    a[0] = cadd(t, a[1]);
    a[1] = csub(t, a[1]);
  }
};

template <bool FWD, typename T2> struct Dft<3, FWD, T2> {
  __device__ static __forceinline__ void run(T2* a) {
    using T = decltype(T2::x);
    const T c = (T)0.86602540378443864676;  // sqrt(3)/2
    T2 s = cadd(a[1], a[2]);
    T2 d = csub(a[1], a[2]);
    T2 m = mk<T2>(a[0].x - (T)0.5 * s.x, a[0].y - (T)0.5 * s.y);
    T2 jd = mul_mi<FWD>(mk<T2>(c * d.x, c * d.y));   // -+ i sqrt(3)/2 d
    a[0] = cadd(a[0], s);
    a[1] = cadd(m, jd);
    a[2] = csub(m, jd);
  }
};

template <bool FWD, typename T2> struct Dft<4, FWD, T2> {
  __device__ static __forceinline__ void run(T2* a) {
    T2 t0 = cadd(a[0], a[2]), t1 = csub(a[0], a[2]);
    T2 t2 = cadd(a[1], a[3]), t3 = mul_mi<FWD>(csub(a[1], a[3]));
    a[0] = cadd(t0, t2);
    a[2] = csub(t0, t2);
    a[1] = cadd(t1, t3);
    a[3] = csub(t1, t3);
  }
};

template <bool FWD, typename T2> struct Dft<8, FWD, T2> {
  __device__ static __forceinline__ void run(T2* a) {
    using T = decltype(T2::x);
    T2 e[4] = {a[0], a[2], a[4], a[6]};
    T2 o[4] = {a[1], a[3], a[5], a[7]};
    Dft<4, FWD, T2>::run(e);
    Dft<4, FWD, T2>::run(o);
    const T s = (T)0.70710678118654752440;
    // o1 *= W8, o2 *= W8^2 = -+i, o3 *= W8^3
    T2 o1 = FWD ? mk<T2>(s * (o[1].x + o[1].y), s * (o[1].y - o[1].x))
                : mk<T2>(s * (o[1].x - o[1].y), s * (o[1].y + o[1].x));
    T2 o2 = mul_mi<FWD>(o[2]);
    T2 o3 = FWD ? mk<T2>(s * (o[3].y - o[3].x), -s * (o[3].x + o[3].y))
                : mk<T2>(-s * (o[3].x + o[3].y), s * (o[3].x - o[3].y));
    a[0] = cadd(e[0], o[0]);
    a[4] = csub(e[0], o[0]);
    a[1] = cadd(e[1], o1);
    a[5] = csub(e[1], o1);
    a[2] = cadd(e[2], o2);
    a[6] = csub(e[2], o2);
    a[3] = cadd(e[3], o3);
    a[7] = csub(e[3], o3);
  }
};

// R = P Q: P-point transforms over n1 of element Q n1 + n2, factors W_R^{n2 k1},
// Q-point transforms over n2; output k1 + P k2
template <int P, int Q, bool FWD, typename T2> struct DftPQ {
  __device__ static __forceinline__ void run(T2* a) {
    T2 y[Q][P];
    sfor<0, Q>([&](auto N2) {
      constexpr int n2 = N2;
#pragma unroll
      for (int n1 = 0; n1 < P; ++n1) y[n2][n1] = a[Q * n1 + n2];
      Dft<P, FWD, T2>::run(y[n2]);
    });
    sfor<0, P>([&](auto K1) {
      constexpr int k1 = K1;
      T2 u[Q];
      sfor<0, Q>([&](auto N2) {
        constexpr int n2 = N2;
        u[n2] = mul_w<P * Q, n2 * k1, FWD>(y[n2][k1]);
      });
      Dft<Q, FWD, T2>::run(u);
#pragma unroll
      for (int k2 = 0; k2 < Q; ++k2) a[k1 + P * k2] = u[k2];
    });
  }
};
template <bool FWD, typename T2> struct Dft<6, FWD, T2> : DftPQ<2, 3, FWD, T2> {};
template <bool FWD, typename T2> struct Dft<12, FWD, T2> : DftPQ<4, 3, FWD, T2> {};
template <bool FWD, typename T2> struct Dft<16, FWD, T2> : DftPQ<4, 4, FWD, T2> {};

// Padded LDS layout of a line held contiguously: element j sits at
// j + (j >> pad_shift<T>()), one pad per pad_run<T>() elements: 16 for c64
// lines, 8 for c128 lines (the run with the fewest bank conflicts for each
// element size).  The stages access a line at strides R and M; the pads spread
// every such group of lanes over distinct banks.
template <typename T> __host__ __device__ constexpr int pad_shift() { return sizeof(T) == 4 ? 4 : 3; }
template <typename T> __host__ __device__ constexpr int pad_run() { return 1 << pad_shift<T>(); }
template <typename T> __host__ __device__ constexpr int lpad(int j) { return j + (j >> pad_shift<T>()); }
// LDS elements a padded line (or twiddle table) of length N occupies
template <typename T> __host__ __device__ constexpr int padded_len(int N) { return N + (N >> pad_shift<T>()) + 1; }
// Index shortcuts of a padded stage: b + r B may be taken as lpad(b) + lpad(r B)
// when B is a multiple of the pad run; the elements base + r Ns of a butterfly
// (base = (b / Ns) Ns R + b % Ns) as lpad(base) + lpad(r Ns) when Ns is, or as
// lpad(base) + r when Ns = 1 and R divides the pad run (base + r then never
// carries into the pad count).
template <typename T> __host__ __device__ constexpr bool read_split(int B) { return B % pad_run<T>() == 0; }
template <typename T> __host__ __device__ constexpr bool write_split(int Ns, int R) {
  return read_split<T>(Ns) || (Ns == 1 && pad_run<T>() % R == 0);
}
// The same base + r Ns where Ns divides the pad run and Ns R is a multiple of
// it: b % Ns never carries, so the element is at lpad(base) + lpad(r Ns).
template <typename T> __host__ __device__ constexpr bool digit_split(int Ns, int R) {
  return pad_run<T>() % Ns == 0 && (Ns * R) % pad_run<T>() == 0;
}

// LDS index of element a of a butterfly whose first element is `base`.
// LS = 0: the line is contiguous from lbase in the padded layout; LS > 0: its
// elements sit LS apart from lbase (lines side by side).
template <typename T, int R, int M, int LS>
__host__ __device__ __forceinline__ int lds_at(int lbase, int base, int a) {
  if constexpr (LS > 0) return lbase + (base + a * M) * LS;
  else if constexpr (write_split<T>(M, R)) return lbase + lpad<T>(base) + (M == 1 ? a : lpad<T>(a * M));
  else if constexpr (digit_split<T>(M, R)) return lbase + lpad<T>(base) + lpad<T>(a * M);
  else return lbase + lpad<T>(base + a * M);
}

// Hand-over of LDS data between the threads of a line.  WAVE: they sit in one
// wavefront, whose LDS instructions execute in order, so only the compiler has
// to keep the order; otherwise a workgroup barrier.
template <bool WAVE> __device__ __forceinline__ void line_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// A thread's place in its line.
struct LineCtx {
  int tl;        // thread index within the line
  int lbase;     // LDS element offset of the line
  bool valid;    // the line exists
};

// v *= W^{+-}: factors between stages s and s + 1 (W_{M R}^{b k} for element k of butterfly j)
template <typename T, int N, int s, bool FWD>
__device__ __forceinline__ void twiddle(c_t<T>* v, int j, const c_t<T>* tw) {
  using St = Stage<N, s>;
  const int b = j % St::M;
#pragma unroll
  for (int k = 1; k < St::R; ++k) {
    c_t<T> w = tw[lpad<T>(b * k * (N / (St::M * St::R)))];
    if (!FWD) w.y = -w.y;
    v[k] = cmul(v[k], w);
  }
}

// What happens to the frequencies between the two directions: apply<N, INV>(v, j)
// gets the outputs v of butterfly j of the last forward stage (frequencies
// freq(j, k)) and, with INV, leaves there what the inverse transform starts from.

// L_a: times lambda^2 / n; adds <Z, L_a Z> = sum lambda^2/n |Z^|^2 (Parseval) to pars.
template <typename T> struct LambdaScale {
  T lamc, invn;
  double& pars;
  template <int N, bool INV> __device__ __forceinline__ void apply(c_t<T>* v, int j) const {
    using St = Stage<N, make_plan(N).S - 1>;
#pragma unroll
    for (int k = 0; k < St::R; ++k) {
      const int f = St::freq(j, k);
      const int p = f < N / 2 ? f : f - N;
      const T lam = lamc * (T)p;
      const T sc = lam * lam * invn;
      pars += (double)sc * (double)cabs2(v[k]);
      if (INV) v[k] = cscale(v[k], sc);
    }
  }
};

// Stages s .. S-1 forward, the scaling, and (INV) the same stages inverse, on
// lines whose stage s input is in LDS (handed over); the result is left there.
template <typename T, int N, int s, int LS, bool WAVE, bool INV, typename Scale>
__device__ __forceinline__ void inner_stages(c_t<T>* lds, const c_t<T>* tw, const LineCtx& lc, const Scale& scale) {
  using T2 = c_t<T>;
  using St = Stage<N, s>;
  constexpr bool kLast = s == St::S - 1;
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    const int j = lc.tl + i * St::T;
    if (lc.valid && St::has(j)) {
      T2 v[St::R];
      const int base = St::base(j);
#pragma unroll
      for (int a = 0; a < St::R; ++a) v[a] = lds[lds_at<T, St::R, St::M, LS>(lc.lbase, base, a)];
      Dft<St::R, true, T2>::run(v);
      if constexpr (kLast) {
        scale.template apply<N, INV>(v, j);
        if constexpr (INV) Dft<St::R, false, T2>::run(v);
      } else {
        twiddle<T, N, s, true>(v, j, tw);
      }
      if constexpr (!kLast || INV) {
#pragma unroll
        for (int a = 0; a < St::R; ++a) lds[lds_at<T, St::R, St::M, LS>(lc.lbase, base, a)] = v[a];
      }
    }
  }
  if constexpr (!kLast) {
    line_sync<WAVE>();
    inner_stages<T, N, s + 1, LS, WAVE, INV>(lds, tw, lc, scale);
    if constexpr (INV) {
      line_sync<WAVE>();
#pragma unroll
      for (int i = 0; i < St::NB; ++i) {
        const int j = lc.tl + i * St::T;
        if (lc.valid && St::has(j)) {
          T2 v[St::R];
          const int base = St::base(j);
#pragma unroll
          for (int a = 0; a < St::R; ++a) v[a] = lds[lds_at<T, St::R, St::M, LS>(lc.lbase, base, a)];
          twiddle<T, N, s, false>(v, j, tw);
          Dft<St::R, false, T2>::run(v);
#pragma unroll
          for (int a = 0; a < St::R; ++a) lds[lds_at<T, St::R, St::M, LS>(lc.lbase, base, a)] = v[a];
        }
      }
    }
  }
}

// Forward transform, `scale`, inverse transform of a line whose stage 0 elements
// the thread holds: v[i][a] is element tl + i T + a M (natural order) on entry
// and, with INV, the same element of the result on return; without, the line
// goes no further than scale.  LDS may be written
// on entry (the caller has handed over whatever it held).
template <typename T, int N> using LineRegs = c_t<T>[Stage<N, 0>::NB][Stage<N, 0>::R];
template <typename T, int N, int LS, bool WAVE, bool INV, typename Scale>
__device__ __forceinline__ void line_apply(LineRegs<T, N>& v, c_t<T>* lds, const c_t<T>* tw, const LineCtx& lc,
                                           const Scale& scale) {
  using T2 = c_t<T>;
  using St = Stage<N, 0>;
  if constexpr (St::S == 1) {
    if (lc.valid && lc.tl == 0) {
      Dft<St::R, true, T2>::run(v[0]);
      scale.template apply<N, INV>(v[0], 0);
      if constexpr (INV) Dft<St::R, false, T2>::run(v[0]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < St::NB; ++i) {
      const int j = lc.tl + i * St::T;
      if (lc.valid && St::has(j)) {
        Dft<St::R, true, T2>::run(v[i]);
        twiddle<T, N, 0, true>(v[i], j, tw);
#pragma unroll
        for (int a = 0; a < St::R; ++a) lds[lds_at<T, St::R, St::M, LS>(lc.lbase, j, a)] = v[i][a];
      }
    }
    line_sync<WAVE>();
    inner_stages<T, N, 1, LS, WAVE, INV>(lds, tw, lc, scale);
    if constexpr (INV) {
      line_sync<WAVE>();
#pragma unroll
      for (int i = 0; i < St::NB; ++i) {
        const int j = lc.tl + i * St::T;
        if (lc.valid && St::has(j)) {
#pragma unroll
          for (int a = 0; a < St::R; ++a) v[i][a] = lds[lds_at<T, St::R, St::M, LS>(lc.lbase, j, a)];
          twiddle<T, N, 0, false>(v[i], j, tw);
          Dft<St::R, false, T2>::run(v[i]);
        }
      }
    }
  }
}

constexpr int ab_batch(int n) { return n >= 96 ? 16 : 8; }

// Projection coefficients of the HVP (Lemma 4.1 with the measured Gram
// system): sums slots 0 and 1 of the x pass's partials (ab.n per slot,
// ab.stride apart) in a fixed order over the workgroup, solves the 2x2 Gram
// system with the set point's component norms ab.gram and returns the
// coefficients in c[0..1] (every thread); res: also stored in ab.res[32..33].
template <int U> __device__ inline void ab_coeffs(const AbSrc& ab, int F, bool store, double* c) {
  __shared__ double red2[2][1024 / kWave];
  __shared__ double cf[2];
  const int t = threadIdx.x;
  double s0 = 0.0, s1 = 0.0;
  // One workgroup beside a pass that fills HBM waits long for each batch of loads,
  // and outlasted the pass with 8 per slot (spin-3 128^3, 16384 partials: y pass 126 ->
  // 121 us, product 490 -> 482, c64 245 -> 235).  U: 16 where the line's own registers
  // are there for them, 8 below (16 costs the c64 pass of length 48 wavefronts, 11.5 ->
  // 12.3 us).  The rest in batches of 4 (clamped addresses: no load waits for a branch).
  const int bd = blockDim.x, n = ab.n;
  int b = t;
  auto batch = [&](auto u_) {
    constexpr int B = decltype(u_)::value;
    double p0[B], p1[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int i = b + u * bd < n ? b + u * bd : n - 1;
      p0[u] = ab.part[i];
      p1[u] = ab.part[ab.stride + i];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      s0 += b + u * bd < n ? p0[u] : 0.0;
      s1 += b + u * bd < n ? p1[u] : 0.0;
    }
    b += B * bd;
  };
  while (b + (U - 1) * bd < n) batch(std::integral_constant<int, U>{});
  while (b < n) batch(std::integral_constant<int, 4>{});
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  if (t % kWave == 0) {
    red2[0][t / kWave] = s0;
    red2[1][t / kWave] = s1;
  }
  __syncthreads();
  if (t == 0) {
    double w0 = 0.0, w1 = 0.0;
    for (int w = 0; w < ((int)blockDim.x + kWave - 1) / kWave; ++w) {
      w0 += red2[0][w];
      w1 += red2[1][w];
    }
    double a11 = 0, a12 = 0, a22 = 0;
    for (int q = 0; q < 2 * F + 1; ++q) {
      const double l = F - q;
      a11 += ab.gram[q];
      a12 += l * ab.gram[q];
      a22 += l * l * ab.gram[q];
    }
    const double det = a11 * a22 - a12 * a12;
    cf[0] = (a22 * w0 - a12 * w1) / det;
    cf[1] = (a11 * w1 - a12 * w0) / det;
    if (store) {
      ab.res[32] = cf[0];
      ab.res[33] = cf[1];
    }
  }
  __syncthreads();
  c[0] = cf[0];
  c[1] = cf[1];
}

// Element at a byte offset from a pointer that is uniform over the wavefront:
// one 32-bit register per address (a component is at most 512^3 c128 values,
// 2^31 bytes).
template <typename T2> __device__ __forceinline__ const T2& at(const T2* base, unsigned off) {
  return *reinterpret_cast<const T2*>(reinterpret_cast<const char*>(base) + off);
}
template <typename T2> __device__ __forceinline__ T2& at(T2* base, unsigned off) {
  return *reinterpret_cast<T2*>(reinterpret_cast<char*>(base) + off);
}

// ---------------------------------------------------------------- axis pass
// An axis pass is bound by HBM (read Z and W, write W; plus X with the
// projection) once its values are in flight early enough, which the register
// plan gives: up to 16 loads of a thread are issued before the first is used,
// and acc and X are read in chunks ahead of the stores (reading acc between the
// stores, which may alias it, serialises them: 150 us for the first row below).
// Measured at spin-3 128^3 (a copy kernel reaches 5.7 TB/s on these sizes):
//   c128 y pass (705 MB) 124 -> 120 us, z pass with projection (940 MB) 171 -> 170;
//   c64 y pass 65 -> 62 us, z pass 89 -> 80;  2D 256^2 spin-2 c128 y pass 13.3 -> 9.5.
//
// Tile: strided lines (y, z) are taken LPB neighbours side by side, so that
// LPB lanes read one contiguous segment, the threads of a line LPB lanes apart;
// contiguous lines (x) have their threads side by side.  Segments of 16 values:
// with 8 c128 values (128 B) the 128^3 passes take 131 and 187 us, as strides
// that are powers of two then use fewer memory channels at a time; 32 c64
// values measure as 16.  Lines of two or more wavefronts' worth per 16 (n >= 192,
// c128) take 8: twice the workgroups on small grids (256^2: 9.5 against 10.6 us).
template <typename T, int N, bool CONTIG> struct AxGeo {
  static constexpr int TPL = make_plan(N).T;
  static constexpr int SEG = sizeof(T) == 8 && TPL > 8 ? 8 : 16;
  static constexpr int LPB = TPL > 16 ? (CONTIG && TPL == 64 ? 1 : 4)      // 384, 512: at most 256 threads
                           : CONTIG || SEG * TPL < 64 ? 64 / TPL : SEG;
  static constexpr int THREADS = ((LPB * TPL + 63) / 64) * 64;
  static constexpr bool kWave = CONTIG ? 64 % TPL == 0 : LPB * TPL <= 64;
  static constexpr int LSTR = padded_len<T>(N);
  static constexpr int TILE = CONTIG ? LPB * LSTR : LPB * N;   // LDS elements of a tile
};

// What an axis pass leaves.  LAP_SUM: the Parseval sum only (no inverse
// transform, no output); LAP_ACC: out and the sum; LAP_FULL: also ||out||^2 of
// the workgroup in the slot after the sum's, and out in c64 at out32 instead of
// at out where out32 is given.
enum LapMode { LAP_ACC = 0, LAP_SUM = 1, LAP_FULL = 2 };

// One axis pass over tile `tile` (LPB lines of one component): out = acc +
// L_a(in) [- (coef[0] + coef[1] l) X], with the Parseval sum <in, L_a in> of
// the workgroup in part[slot * stride + blk] when part != null.  GROUPS tiles
// share a workgroup (batched launches).
template <typename T, int N, bool CONTIG, int GROUPS = 1, int MODE = LAP_ACC>
__device__ __forceinline__ void lap_body(const c_t<T>* __restrict__ in, const c_t<T>* acc, c_t<T>* out,
                                         const c_t<T>* __restrict__ twg, int inner, T lamc, int F, size_t npts,
                                         const c_t<T>* __restrict__ X, const double* __restrict__ coef,
                                         double* __restrict__ part, size_t stride, int slot, long blk,
                                         const double* skip, const AbSrc& ab, float2* out32 = nullptr) {
  if (skip && *skip != 0.0) return;   // uniform over the workgroup
  using T2 = c_t<T>;
  using G = AxGeo<T, N, CONTIG>;
  using St = Stage<N, 0>;
  constexpr int TPL = G::TPL, LPB = G::LPB;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T2* tw = reinterpret_cast<T2*>(smem_raw);
  // (a tile's threads are whole wavefronts)
  const int grp = GROUPS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / G::THREADS) : 0;
  const int t = GROUPS > 1 ? (int)threadIdx.x % G::THREADS : (int)threadIdx.x;
  T2* lds = tw + padded_len<T>(N) + grp * G::TILE;
  if constexpr (St::S > 1)
    for (int m = threadIdx.x; m < N; m += blockDim.x) tw[lpad<T>(m)] = twg[m];

  const unsigned lpc = (unsigned)(npts / N);    // lines per component: a tile never straddles two
  const unsigned tpc = (lpc + LPB - 1) / LPB;
  const unsigned tile = (unsigned)blk * GROUPS + grp;
  const int comp = (int)(tile / tpc);
  const int ln = CONTIG ? t / TPL : t % LPB;
  const unsigned line = (tile - (unsigned)comp * tpc) * LPB + ln;   // within the component
  LineCtx lc;
  lc.tl = CONTIG ? t % TPL : t / LPB;
  lc.lbase = CONTIG ? ln * G::LSTR : ln;
  lc.valid = ln < LPB && lc.tl < TPL && comp < 2 * F + 1 && line < lpc;
  // byte offsets within the component: of the thread's first element, and along the line
  const unsigned gs = CONTIG ? 1u : (unsigned)inner;
  const unsigned goff = (unsigned)sizeof(T2) * ((CONTIG ? line * N : line / gs * (N * gs) + line % gs) + lc.tl * gs);
  const unsigned gstep = (unsigned)sizeof(T2) * gs;
  const size_t cbase = (size_t)comp * npts;
  const T invn = T(1) / T(N);

  LineRegs<T, N> v;
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    const int j = lc.tl + i * TPL;
    if (lc.valid && St::has(j)) {
#pragma unroll
      for (int a = 0; a < St::R; ++a) v[i][a] = at(in + cbase, goff + (i * TPL + a * St::M) * gstep);
    }
  }
  double c0 = 0.0, c1 = 0.0;
  if (X && ab.part) {   // uniform: the coefficients from the x pass's partials
    double cf[2];
    ab_coeffs<ab_batch(N)>(ab, F, blk == 0, cf);
    c0 = cf[0];
    c1 = cf[1];
  } else if (X) {
    c0 = coef[0];
    c1 = coef[1];
  }
  const T pc = (T)(c0 + c1 * (double)(F - comp));   // (0 without a projection)
  double pars = 0.0;
  if constexpr (St::S > 1) __syncthreads();   // the twiddle table
  line_apply<T, N, CONTIG ? 0 : LPB, G::kWave, MODE != LAP_SUM>(v, lds, tw, lc, LambdaScale<T>{lamc, invn, pars});
  double sums[MODE == LAP_FULL ? 2 : 1];
  sums[0] = pars;
  if constexpr (MODE == LAP_FULL) sums[1] = 0.0;
  // (acc may be out: its values are read ahead of the stores, a chunk at a time)
  constexpr int CH = St::R % 8 == 0 ? 8 : St::R % 6 == 0 ? 6 : St::R;
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    if (MODE != LAP_SUM && lc.valid && St::has(lc.tl + i * TPL)) {
#pragma unroll
      for (int a0 = 0; a0 < St::R; a0 += CH) {
        T2 w[CH], xv[CH];
#pragma unroll
        for (int a = 0; a < CH; ++a) {
          const unsigned g = goff + (i * TPL + (a0 + a) * St::M) * gstep;
          w[a] = acc ? at(acc + cbase, g) : mk<T2>(0, 0);
          xv[a] = X ? at(X + cbase, g) : mk<T2>(0, 0);
        }
#pragma unroll
        for (int a = 0; a < CH; ++a) {
          const unsigned g = goff + (i * TPL + (a0 + a) * St::M) * gstep;
          T2 o = cadd(w[a], v[i][a0 + a]);
          o.x -= pc * xv[a].x;
          o.y -= pc * xv[a].y;
          if constexpr (MODE == LAP_FULL) {
            sums[1] += (double)cabs2(o);
            if (out32) at(out32 + cbase, g / (sizeof(T2) / sizeof(float2))) = mk<float2>((float)o.x, (float)o.y);
            else at(out + cbase, g) = o;
          } else {
            at(out + cbase, g) = o;
          }
        }
      }
    }
  }
  if (part) block_partials_any(sums, part + (size_t)slot * stride, stride, blk);
}

#define GPE_SIZES(M) M(4) M(6) M(8) M(12) M(16) M(24) M(32) M(48) M(64) M(96) M(128) M(192) M(256) M(384) M(512)

// Tiles (workgroups) of an axis pass over K components of npts points.
template <typename T, int N, bool CONTIG> constexpr long ax_tiles(int K, size_t npts) {
  return (long)K * (((long)(npts / N) + AxGeo<T, N, CONTIG>::LPB - 1) / AxGeo<T, N, CONTIG>::LPB);
}

// ---------------------------------------------------------------- fused x pass
// Fused x pass of the Hessian-vector product: RPB x-rows, all K components.
// Geometry VAR: rows per workgroup for about one wavefront (0), two (1, the
// default) or four (2); XVAR_LATENCY: one row and a thread for each of
// its points, for grids whose few workgroups are bound by a thread's chain of
// FP64 operations (the threads beyond the lines' idle during the transform).  At
// n = 128, K = 7 a variant-0 workgroup is one wavefront that owns one row of every
// component: 56 lanes hold 16 values each for the transform, 64 lanes two points
// each for the pointwise terms.
//
// Bound by its 29 streams of HBM traffic (4 fields and V; 5.0 TB/s of the copy
// rate's 5.7 for this pattern) in c128 and by those and VALU issue in c64.  The
// pointwise terms come first, while every operand is read once, and their
// result q stays in registers; only the row of Z passes through LDS, so no
// second copy of Z is kept there and twice the rows fit a CU.  The kernel has
// no row loop: hoisted out of one, the spin constants fill the registers (256,
// with spills).  At least 2 (c128) and 4 (c64) wavefronts per SIMD: 3 in c128
// spill 70 registers.  Measured (c128, c64):
//   spin-3 128^3 247 -> 194 us, 140 -> 102;  spin-1 256 x 256 x 64 212 -> 165, 92 -> 82;
//   spin-2 96^3 79 -> 55 us, 41 -> 32;  spin-2 256^2 (one row) 12.6 -> 10.3, 10.2 -> 8.0.
// Operands of the next point fetched ahead gain nothing (spin-1 256 x 256 x 64 167 ->
// 166, 88 -> 87) and spill in c64 from K = 5 on (96^3 32 -> 43).
constexpr int XVAR_LATENCY = 3;
template <int N, int K, int VAR = 1> struct XGeo {
  static constexpr int TPL = make_plan(N).T;
  static constexpr int WANT = VAR == 0 ? 64 : VAR == 1 ? 128 : 256;
  static constexpr int RPB = VAR == XVAR_LATENCY ? (N >= 64 ? 1 : 64 / N)
                                                 : (WANT / (K * TPL) >= 1 ? WANT / (K * TPL) : 1);
  static constexpr int LINES = RPB * K;
  static constexpr int WORK = VAR == XVAR_LATENCY && RPB * N > LINES * TPL ? RPB * N : LINES * TPL;
  static constexpr int THREADS = ((WORK + 63) / 64) * 64;
  static constexpr int PPT = (RPB * N + THREADS - 1) / THREADS;   // points per thread
  static constexpr bool kWave = 64 % TPL == 0;
  // LDS: the padded twiddle table, then LINES padded lines
  template <typename T> static constexpr int lstr() { return padded_len<T>(N); }
  template <typename T> static constexpr size_t lds_elems() { return (size_t)lstr<T>() * (1 + LINES); }
};

// A whole product in one workgroup (1D grids: one row is the grid): the sums, the
// projection and the post-operations happen where W is still in registers and LDS.
struct OneArgs {
  double* gram = nullptr;     // component norms of the set point
  double* res = nullptr;
  double* mirror = nullptr;   // see finalize
  int post = POST_NONE;       // after the projection's Gram solve
  bool proj = false;
};

template <typename T, int N, int F, int VAR, bool ONE = false>
__device__ __forceinline__ void xpass_body(const c_t<T>* __restrict__ X, const c_t<T>* __restrict__ Z,
                                           const c_t<T>* __restrict__ Y, const T* __restrict__ V,
                                           c_t<T>* __restrict__ W, const c_t<T>* __restrict__ twg, long nrows,
                                           size_t npts, T lamc, const PwParams& p, double* __restrict__ part,
                                           size_t stride, long blk, const double* skip,
                                           const OneArgs& one = OneArgs{}) {
  if (skip && *skip != 0.0) return;   // uniform over the workgroup
  using T2 = c_t<T>;
  constexpr int K = 2 * F + 1;
  using G = XGeo<N, K, VAR>;
  using St = Stage<N, 0>;
  constexpr int TPL = G::TPL, RPB = G::RPB, LINES = G::LINES, PPT = G::PPT;
  constexpr int LSTR = G::template lstr<T>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T2* tw = reinterpret_cast<T2*>(smem_raw);
  T2* lds = tw + LSTR;
  const int t = threadIdx.x;
  if constexpr (St::S > 1)
    for (int m = t; m < N; m += blockDim.x) tw[lpad<T>(m)] = twg[m];
  const T invn = T(1) / T(N);
  T zcoef[K];
#pragma unroll
  for (int i = 0; i < K; ++i) zcoef[i] = (T)p.zc[i];
  double acc[7] = {0, 0, 0, 0, 0, 0, 0};

  const long row0 = blk * RPB;
  // ---- pointwise Hessian terms q of this thread's points; the rows of Z go
  // to LDS for the transform.  Per point the partial sums run over the K
  // components in the work precision; the sums over points accumulate in FP64.
  T2 q[PPT][K];
  const size_t r0 = (size_t)row0 * N;   // (the points of the row block are contiguous)
  const unsigned np = (unsigned)(nrows - row0 < RPB ? nrows - row0 : RPB) * N;
#pragma unroll
  for (int pp = 0; pp < PPT; ++pp) {
    const unsigned pt = t + pp * G::THREADS;
    if (t < G::THREADS && pt < np) {
      T2 x[K], z[K], y[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        z[i] = at(Z + r0 + i * npts, pt * (unsigned)sizeof(T2));
        x[i] = at(X + r0 + i * npts, pt * (unsigned)sizeof(T2));
      }
      if (Y) {
#pragma unroll
        for (int i = 0; i < K; ++i) y[i] = at(Y + r0 + i * npts, pt * (unsigned)sizeof(T2));
      } else {
#pragma unroll
        for (int i = 0; i < K; ++i) y[i] = mk<T2>(0, 0);
      }
      const T vj = at(V + r0, pt * (unsigned)sizeof(T));
      T s_xw = 0, s_lxw = 0, s_xz = 0, s_lxz = 0, s_zq = 0, s_zz = 0;
#pragma unroll
      for (int i = 0; i < K; ++i) {
        lds[(i * RPB + pt / N) * LSTR + lpad<T>(pt % N)] = z[i];
        const T c = cdotr(y[i], z[i]);     // <(LX)_i, Z_i> = <X_i, (LZ)_i>
        const T xz = cdotr(x[i], z[i]);
        s_xw += c;
        s_lxw += T(F - i) * c;
        s_xz += xz;
        s_lxz += T(F - i) * xz;
        s_zz += cabs2(z[i]);
      }
      hvp_point<T, F>(x, z, vj, p, zcoef, [&](int i, T2 qi) {
        q[pp][i] = qi;
        const T xq = cdotr(x[i], qi);
        s_xw += xq;
        s_lxw += T(F - i) * xq;
        s_zq += cdotr(z[i], qi);
      });
      acc[0] += (double)s_xw;
      acc[1] += (double)s_lxw;
      acc[2] += (double)s_xz;
      acc[3] += (double)s_lxz;
      acc[4] += (double)s_zq;
      acc[5] += (double)s_zz;
    }
    // one point at a time: interleaving several would hold all their operands at once
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();   // the rows of Z (and the twiddle table)

  // ---- L_x Z for the RPB rows of every component, in place in LDS
  LineCtx lc;
  const int ls = t / TPL;                 // line slot = comp * RPB + row
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
  line_apply<T, N, 0, G::kWave, true>(v, lds, tw, lc, LambdaScale<T>{lamc, invn, acc[6]});
#pragma unroll
  for (int i = 0; i < St::NB; ++i) {
    const int j = lc.tl + i * TPL;
    if (lc.valid && St::has(j)) {
#pragma unroll
      for (int a = 0; a < St::R; ++a) lds[lds_at<T, St::R, St::M, 0>(lc.lbase, j, a)] = v[i][a];
    }
  }
  __syncthreads();

  // ---- ONE: sums, Gram solve and post-operations in this workgroup
  __shared__ double sum[ONE ? 8 : 1], state[ONE ? 64 : 1];
  if constexpr (ONE) {
    if (t < 64) state[t] = one.res[t];
    block_sums(acc, [&](int k, double s) { sum[k] = s; });
    __syncthreads();
    if (t == 0) {
      if (one.proj) finalize_post(sum, 7, state, one.res, POST_HVP_AB, F, nullptr, one.gram);
      if (one.post != POST_NONE) finalize_post(sum, 7, state, one.res, one.post, F, nullptr, one.gram);
    }
    __syncthreads();
    if (one.mirror && t < 64) one.mirror[t] = state[t];
  }

  // ---- W = L_x Z + q [- (alpha_w + beta_w l) X]
#pragma unroll
  for (int pp = 0; pp < PPT; ++pp) {
    const unsigned pt = t + pp * G::THREADS;
    if (t < G::THREADS && pt < np) {
#pragma unroll
      for (int i = 0; i < K; ++i) {
        T2 w = cadd(lds[(i * RPB + pt / N) * LSTR + lpad<T>(pt % N)], q[pp][i]);
        if constexpr (ONE) {
          if (one.proj) {
            const T c = (T)(state[32] + state[33] * (double)(F - i));
            const T2 xv = at(X + r0 + i * npts, pt * (unsigned)sizeof(T2));
            w.x -= c * xv.x;
            w.y -= c * xv.y;
          }
        }
        at(W + r0 + i * npts, pt * (unsigned)sizeof(T2)) = w;
      }
    }
  }
  if constexpr (!ONE) block_partials_any<7>(acc, part, stride, blk);
}

}  // namespace gpe
