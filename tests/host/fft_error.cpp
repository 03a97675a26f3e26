// FP32 rounding error of the transforms of csrc/fft.hpp beside that of the
// textbook stages (products with w^(r k), then the untwiddled DFT), against
// FP64.  Prints per configuration: N, direction, schedule, RMS error and the
// textbook's, both relative to the RMS output.
#include "lanes.hpp"

#include <cstdio>
#include <random>

#include "fft.hpp"

using namespace ttsh;

template <class T>
static std::vector<C2<T>> waves(int N) {
  std::vector<C2<T>> w(N);
  for (int j = 0; j < N; ++j) w[j] = mk((T)std::cos(2 * M_PI * j / N), (T)-std::sin(2 * M_PI * j / N));
  return w;
}

template <class T>
static std::vector<C2<T>> table(int N) {
  std::vector<C2<T>> w(N / 2);
  for (int j = 0; j < N / 2; ++j) w[j] = fft_factor<T>(j, N);
  return w;
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

template <int N, int DIR, int SCH>
void one() {
  constexpr int TT = N / kFftE, COUNT = N <= 512 ? 32768 / N : 32;
  const auto wf = waves<float>(N);
  const auto wd = waves<double>(N);
  const auto tf = table<float>(N);
  std::mt19937_64 gen(N + DIR);
  std::normal_distribution<double> U(0, 1);
  double ours = 0, book = 0, size = 0;
  std::vector<C2<float>> lds(Padded<N, SCH>::value);
  for (int q = 0; q < COUNT; ++q) {
    std::vector<C2<float>> x(N), y(N);
    std::vector<C2<double>> d(N);
    for (int i = 0; i < N; ++i) {
      x[i] = mk((float)U(gen), (float)U(gen));
      d[i] = mk((double)x[i].x, (double)x[i].y);
    }
    lanes::run(TT, false, [&](int t) {
      C2<float> v[1][kFftE];
      for (int e = 0; e < kFftE; ++e) v[0][e] = x[t + e * TT];
      fft<N, DIR, 1, SCH, false>(v, lds.data(), t, tf.data());
      for (int e = 0; e < kFftE; ++e) y[t + e * TT] = v[0][e];
    });
    textbook<N, DIR, SCH>(x, wf);
    textbook<N, DIR, SCH>(d, wd);
    for (int i = 0; i < N; ++i) {
      ours += std::pow(y[i].x - d[i].x, 2) + std::pow(y[i].y - d[i].y, 2);
      book += std::pow(x[i].x - d[i].x, 2) + std::pow(x[i].y - d[i].y, 2);
      size += d[i].x * d[i].x + d[i].y * d[i].y;
    }
  }
  std::printf("%d %d %d %.4e %.4e\n", N, DIR, SCH, std::sqrt(ours / size), std::sqrt(book / size));
}

template <int N>
void both() {
  one<N, -1, kSchedDefault>();
  one<N, +1, kSchedDefault>();
}

int main() {
  both<64>();
  both<128>();
  both<256>();
  both<512>();
  both<1024>();
  both<2048>();
  both<4096>();
  both<8192>();
  one<128, -1, sched_code(4, true)>();
  one<256, +1, sched_code(4, true)>();
  return 0;
}
