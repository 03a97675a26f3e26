// Rounding error of the transforms of csrc/fft.hpp beside that of the textbook
// stages (products with w^(r k), then the untwiddled DFT) with factors rounded
// once, against long double.  Prints per configuration: bits of the type, N,
// direction, schedule, RMS error and the textbook's, both relative to the RMS
// output.
#include "lanes.hpp"

#include <cstdio>
#include <random>

#include "fft.hpp"

using namespace ttsh;
using X = long double;

static C2<X> wave(X turn) {  // e^{-2 pi i turn}
  const X a = 2 * 3.14159265358979323846264338327950288L * turn;
  return mk(cosl(a), -sinl(a));
}

template <class T>
static std::vector<C2<T>> waves(int N) {
  std::vector<C2<T>> w(N);
  for (int j = 0; j < N; ++j) w[j] = cvt<T>(wave((X)j / N));
  return w;
}

template <class T>
static std::vector<C2<T>> table(int N) {
  std::vector<C2<T>> w(N / 2);
  fft_factors(N, w.data());
  return w;
}

// the reference: halves of even and odd elements
static std::vector<C2<X>> exact(const std::vector<C2<X>>& x, int dir) {
  const int n = (int)x.size();
  if (n == 1) return x;
  std::vector<C2<X>> e(n / 2), o(n / 2), y(n);
  for (int i = 0; i < n / 2; ++i) e[i] = x[2 * i], o[i] = x[2 * i + 1];
  e = exact(e, dir);
  o = exact(o, dir);
  for (int i = 0; i < n / 2; ++i) {
    C2<X> w = wave((X)i / n);
    if (dir > 0) w = conj(w);
    const C2<X> t = cmul(o[i], w);
    y[i] = e[i] + t;
    y[i + n / 2] = e[i] - t;
  }
  return y;
}

template <int N, int DIR, int SCH, class T, int P = 1>
void textbook(std::vector<C2<T>>& x, const std::vector<C2<T>>& w) {
  constexpr int R = stage_radix<N, SCH>(P);
  std::vector<C2<T>> y(N);
  for (int i = 0; i < N / R; ++i) {
    const int k = i % P;
    C2<T> u[R];
    for (int r = 0; r < R; ++r) {
      C2<T> f = w[(size_t)r * k * (N / (P * R))], a = x[i + r * (N / R)];
      if (DIR > 0) f = conj(f);
      u[r] = r * k ? mk(fma(a.x, f.x, -(a.y * f.y)), fma(a.x, f.y, a.y * f.x)) : a;
    }
    Dft<R, DIR, T>::run(u);
    for (int r = 0; r < R; ++r) y[(i - k) * R + k + r * P] = u[r];
  }
  x = y;
  if constexpr (P * R < N) textbook<N, DIR, SCH, T, P * R>(x, w);
}

template <class T, int N, int DIR, int SCH>
void one() {
  constexpr int TT = N / kFftE, COUNT = N <= 1024 ? 16384 / N : 8;
  const auto wt = waves<T>(N);
  const auto ft = table<T>(N);
  std::mt19937_64 gen(N + DIR);
  std::normal_distribution<double> U(0, 1);
  X ours = 0, book = 0, size = 0;
  std::vector<C2<T>> lds(Padded<N, SCH>::value);
  for (int q = 0; q < COUNT; ++q) {
    std::vector<C2<T>> x(N), y(N);
    std::vector<C2<X>> d(N);
    for (int i = 0; i < N; ++i) {
      x[i] = mk((T)U(gen), (T)U(gen));
      d[i] = cvt<X>(x[i]);
    }
    lanes::run(TT, false, [&](int t) {
      C2<T> v[1][kFftE];
      for (int e = 0; e < kFftE; ++e) v[0][e] = x[t + e * TT];
      fft<N, DIR, 1, SCH, false>(v, lds.data(), t, ft.data());
      for (int e = 0; e < kFftE; ++e) y[t + e * TT] = v[0][e];
    });
    textbook<N, DIR, SCH>(x, wt);
    d = exact(d, DIR);
    for (int i = 0; i < N; ++i) {
      const C2<X> a = cvt<X>(y[i]) - d[i], b = cvt<X>(x[i]) - d[i];
      ours += a.x * a.x + a.y * a.y;
      book += b.x * b.x + b.y * b.y;
      size += d[i].x * d[i].x + d[i].y * d[i].y;
    }
  }
  std::printf("%d %d %d %d %.4e %.4e\n", (int)sizeof(T) * 8, N, DIR, SCH, (double)sqrtl(ours / size),
              (double)sqrtl(book / size));
}

template <class T, int N>
void both() {
  one<T, N, -1, kSchedDefault>();
  one<T, N, +1, kSchedDefault>();
}
template <class T>
void all() {
  both<T, 64>();
  both<T, 128>();
  both<T, 256>();
  both<T, 512>();
  both<T, 1024>();
  both<T, 2048>();
  both<T, 4096>();
  both<T, 8192>();
  one<T, 128, -1, sched_code(4, true)>();
  one<T, 256, +1, sched_code(4, true)>();
}

int main() {
  all<float>();
  all<double>();
  return 0;
}
