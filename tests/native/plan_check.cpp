// Host check of the line transforms' index arithmetic over the plans the kernels
// use: for every line length, stage, butterfly and element, the LDS index of
// the padded layout with its shortcuts against the index in full (both element
// sizes) and that of lines side by side; every element of a line belongs to
// exactly one butterfly of each stage; a later stage's butterflies stay within
// one output block of the stage before (in place); and the frequencies of the
// last stage's outputs are a permutation, each the digit reversal that the
// stages' strides make of its location.  Prints the number of violations and
// exits non-zero if there are any.
#include <cstdio>
#include <set>
#include <vector>

#include "fft.h"

static long checked = 0, bad = 0, split = 0;
static void expect(bool ok) {
  ++checked;
  bad += !ok;
}

// frequency at location p of a line of N values after the forward stages R[0..S-1]:
// stage s leaves at digit d (stride M) of its block the frequency's digit of weight R[0] .. R[s-1]
static int freq_at(int N, const std::vector<int>& R, int p) {
  int f = 0, w = 1, M = N;
  for (int r : R) {
    M /= r;
    f += w * (p / M);
    p %= M;
    w *= r;
  }
  return f;
}

template <typename T, int N, int s> static void stage() {
  using St = gpe::Stage<N, s>;
  using gpe::lpad;
  constexpr int kLines = 3;
  std::vector<int> seen(N, 0);
  expect(St::R * St::NBF == N && St::NB * St::T >= St::NBF);
  split += (gpe::write_split<T>(St::M, St::R) || gpe::digit_split<T>(St::M, St::R)) ? 1 : 0;
  for (int j = 0; j < St::NBF; ++j) {
    expect(St::has(j));
    const int base = St::base(j);
    for (int a = 0; a < St::R; ++a) {
      const int e = base + a * St::M;
      expect(e >= 0 && e < N);
      ++seen[e];
      expect(base / (St::M * St::R) == e / (St::M * St::R));
      expect((gpe::lds_at<T, St::R, St::M, 0>(7, base, a)) == 7 + lpad<T>(e));
      expect(lpad<T>(e) < gpe::padded_len<T>(N));
      expect((gpe::lds_at<T, St::R, St::M, kLines>(2, base, a)) == 2 + e * kLines);
    }
  }
  for (int n : seen) expect(n == 1);
}

template <typename T, int N, int s = 0> static void stages(std::vector<int> R = {}) {
  stage<T, N, s>();
  using St = gpe::Stage<N, s>;
  R.push_back(St::R);
  if constexpr (s + 1 < St::S) {
    stages<T, N, s + 1>(R);
  } else {
    std::set<int> f;
    for (int j = 0; j < St::NBF; ++j)
      for (int k = 0; k < St::R; ++k) {
        expect(St::freq(j, k) == freq_at(N, R, St::base(j) + k * St::M));
        f.insert(St::freq(j, k));
      }
    expect((int)f.size() == N && *f.begin() == 0 && *f.rbegin() == N - 1);
  }
}

int main() {
#define CHECK(N) stages<float, N>(); stages<double, N>();
  GPE_SIZES(CHECK)
  std::printf("%ld checked, %ld stages with a shortcut, violations %ld\n", checked, split, bad);
  return bad != 0;
}
