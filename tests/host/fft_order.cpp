// The transforms of csrc/fft.hpp with their lanes run one by one between
// fences (lanes.hpp), against the defining sums in FP64.  Prints one line per
// configuration: N, direction, transforms, schedule, one-wavefront workgroup,
// lane order, largest error relative to the largest output.
#include "lanes.hpp"

#include <algorithm>
#include <cstdio>
#include <random>

#include "fft.hpp"

using namespace ttsh;
using C = C2<double>;

static std::vector<C> table(int N) {
  std::vector<C> w(N);
  for (int j = 0; j < N; ++j) w[j] = mk(std::cos(2 * M_PI * j / N), -std::sin(2 * M_PI * j / N));
  return w;
}

static std::vector<C> factors(int N) {
  std::vector<C> w(N / 2);
  fft_factors(N, w.data());
  return w;
}

template <int N, int DIR, int NF, int SCH, bool WAVE, bool KEPT>
void one(bool descending) {
  constexpr int TT = N / kFftE, G = WAVE ? 64 / TT : 1, NT = G * TT;
  constexpr int REG = fft_slots(NF, WAVE) * Padded<N, SCH>::value;
  const std::vector<C> tw = factors(N), wave = table(N);
  std::mt19937_64 gen(7 * N + NF);
  std::uniform_real_distribution<double> U(-1, 1);
  std::vector<C> x((size_t)G * NF * N), y(x.size()), lds((size_t)G * REG);
  for (auto& v : x) v = mk(U(gen), U(gen));
  lanes::run(NT, descending, [&](int tid) {
    const int t = tid % TT, g = tid / TT;
    C v[NF][kFftE];
    for (int f = 0; f < NF; ++f)
      for (int e = 0; e < kFftE; ++e) v[f][e] = x[(size_t)(g * NF + f) * N + t + e * TT];
    if constexpr (KEPT) {
      Factors<N, double, SCH> fac;
      fac.load(tw.data(), t);
      fft<N, DIR, NF, SCH, WAVE>(v, lds.data() + g * REG, t, fac);
    } else {
      fft<N, DIR, NF, SCH, WAVE>(v, lds.data() + g * REG, t, tw.data());
    }
    for (int f = 0; f < NF; ++f)
      for (int e = 0; e < kFftE; ++e) y[(size_t)(g * NF + f) * N + t + e * TT] = v[f][e];
  });
  double err = 0, big = 0;
  for (int q = 0; q < G * NF; ++q)
    for (int m = 0; m < N; ++m) {
      C s = mk(0.0, 0.0);
      for (int n = 0; n < N; ++n) {
        const C w = wave[(size_t)m * n % N];
        s = s + cmul(x[(size_t)q * N + n], DIR > 0 ? conj(w) : w);
      }
      const C d = y[(size_t)q * N + m] - s;
      err = std::max({err, std::fabs(d.x), std::fabs(d.y)});
      big = std::max({big, std::fabs(s.x), std::fabs(s.y)});
    }
  std::printf("%d %d %d %d %d %d %d %.3e\n", N, DIR, NF, SCH, (int)WAVE, (int)KEPT, (int)descending, err / big);
}

template <int N, int SCH, bool WAVE>
void sizes() {
  for (bool d : {false, true}) {
    one<N, -1, 1, SCH, WAVE, false>(d);
    one<N, -1, 2, SCH, WAVE, false>(d);
    one<N, +1, 3, SCH, WAVE, false>(d);
    one<N, -1, 3, SCH, WAVE, true>(d);
    one<N, +1, 2, SCH, WAVE, true>(d);
  }
}

int main() {
  sizes<64, kSchedDefault, true>();
  sizes<128, kSchedDefault, true>();
  sizes<256, kSchedDefault, true>();
  sizes<512, kSchedDefault, true>();
  sizes<128, sched_code(3, true), true>();
  sizes<256, sched_code(5, true), true>();
  sizes<64, kSchedDefault, false>();
  sizes<128, kSchedDefault, false>();
  sizes<256, kSchedDefault, false>();
  sizes<1024, kSchedDefault, false>();
  return 0;
}
