// Workgroup-level Stockham FFT staged through LDS, for gfx950.
//
// One transform of length N (64..8192, a power of two) is carried by TT = N/8
// threads of a workgroup; thread t holds the 8 elements t + e*TT (e = 0..7)
// in registers.  Each stage of radix R (8, and one 4 or 2) reads its butterfly
// inputs x[i + r*N/R] from exactly those registers, takes the radix-R DFT of
// their products with w^(r*k) (k = i mod P, P the product of the earlier
// radices; w^(r*k) inside the DFT's own butterflies, see DftTw) and scatters
// the outputs to y[(i-k)R + k + rP] (Stockham autosort, decimation in time; Van
// Loan, Computational Frameworks for the FFT, ch. 1.7).  Because the input
// stride N/R is the same in every stage, the scatter is followed by a gather of
// t + e*TT, and in the last stage (P = N/R) the scatter target is t + e*TT
// itself, so the output lands in the registers that held the input, in natural
// order.  A transform therefore costs (#stages - 1) LDS round trips and needs
// no bit reversal.
//
// NF independent transforms that share the same threads are processed
// together.  At most TTSH_FFT_SLOTS of them occupy LDS at a time: with as many
// slots as transforms one barrier pair per stage serves all of them; with
// fewer, the transforms take turns in the slots (one more barrier per extra
// transform and stage), which shrinks the LDS footprint of a transform group
// and lets more waves stay resident on a CU.  One-wavefront workgroups, whose
// barriers cost nothing, use a single slot.
//
// All threads of the workgroup must call these functions (they contain
// workgroup barriers, or wavefront-scope ordering for one-wavefront
// workgroups); threads that carry no useful data just transform zeros.
#pragma once

#include <cmath>

#include "common.hpp"

namespace ttsh {

constexpr int kFftE = 8;  // elements per thread

// Schedule of a transform, one int SCH = 2 PAD + SMALL_FIRST:
//   PAD          the LDS index gets one pad slot every 2^PAD entries (breaks
//                the strided scatter of the stages across banks);
//   SMALL_FIRST  for N not a power of 8, whether the radix left over after
//                the radix-8 stages (2 or 4) runs as the first stage or the
//                last one.
// The default (one slot per 16, small radix last) was the fastest of the
// hand-measured settings on gfx950; the autotuner also tries PAD = 3, 5 and
// the small radix first for the time-step kernels.  The schedule changes
// neither the result's layout nor, for the padding, its arithmetic.
constexpr int sched_code(int pad, bool small_first) { return 2 * pad + (small_first ? 1 : 0); }
constexpr int kSchedDefault = sched_code(4, false);
constexpr int sched_pad(int sch) { return sch >> 1; }
constexpr bool sched_small_first(int sch) { return (sch & 1) != 0; }

template <int SCH = kSchedDefault>
__host__ __device__ constexpr int lds_pad(int j) { return j + (j >> sched_pad(SCH)); }
// lds_pad(j + rP) - lds_pad(j) for j whose remainder modulo P R (a power of
// two) is below P, r < R: the low bits of j and of rP do not overlap, so no
// carry crosses the 2^PAD boundary and the difference is a constant.  The
// accesses of a stage thus share one LDS address and differ by immediate
// offsets, instead of keeping one address register each.
template <int SCH = kSchedDefault>
__host__ __device__ constexpr int lds_step(int rP) { return rP + (rP >> sched_pad(SCH)); }
template <int N, int SCH = kSchedDefault>
struct Padded {
  static constexpr int value = N + (N >> sched_pad(SCH));
};

// radix of the stage that follows stages whose radices multiply to P
template <int N, int SCH>
constexpr int stage_radix(int P) {
  int l2 = 0;
  while ((1 << l2) < N) ++l2;
  const int small = 1 << (l2 % 3);  // 1, 2 or 4
  if (sched_small_first(SCH) && small > 1) return P == 1 ? small : 8;
  const int rem = N / P;
  return rem % 8 == 0 ? 8 : (rem % 4 == 0 ? 4 : 2);
}

#ifndef TTSH_FFT_SLOTS
#define TTSH_FFT_SLOTS 2
#endif
static_assert(TTSH_FFT_SLOTS >= 2, "the slot rotation needs at least two slots");
// LDS regions of Padded<N> entries that NF transforms use during an exchange.
// A one-wavefront tile (wave) needs a single one: its LDS accesses execute in
// issue order, so a transform may overwrite the region as soon as the gather
// of the one before has been issued (lds_sync keeps the compiler to that order).
__host__ __device__ constexpr int fft_slots(int nf, bool wave = false) {
  return wave ? 1 : nf < TTSH_FFT_SLOTS ? nf : TTSH_FFT_SLOTS;
}

// ---- radix-R DFTs, DIR = -1 forward (e^{-2 pi i nk/R}), +1 inverse ---------
template <int DIR, class T>
__device__ __forceinline__ void dft4(C2<T>& a0, C2<T>& a1, C2<T>& a2, C2<T>& a3) {
  const C2<T> t0 = a0 + a2, t1 = a0 - a2, t2 = a1 + a3;
  const C2<T> t3 = mul_i<DIR>(a1 - a3);
  a0 = t0 + t2;
  a2 = t0 - t2;
  a1 = t1 + t3;
  a3 = t1 - t3;
}

template <int R, int DIR, class T>
struct Dft;

template <int DIR, class T>
struct Dft<2, DIR, T> {
  __device__ static __forceinline__ void run(C2<T> (&u)[2]) {
    const C2<T> d = u[0] - u[1];
    u[0] = u[0] + u[1];
    u[1] = d;
  }
};

template <int DIR, class T>
struct Dft<4, DIR, T> {
  __device__ static __forceinline__ void run(C2<T> (&u)[4]) { dft4<DIR>(u[0], u[1], u[2], u[3]); }
};

template <int DIR, class T>
struct Dft<8, DIR, T> {
  __device__ static __forceinline__ void run(C2<T> (&u)[8]) {
    // even / odd halves, then combine with W8^k = e^{DIR 2 pi i k / 8}
    C2<T> e0 = u[0], e1 = u[2], e2 = u[4], e3 = u[6];
    C2<T> o0 = u[1], o1 = u[3], o2 = u[5], o3 = u[7];
    dft4<DIR>(e0, e1, e2, e3);
    dft4<DIR>(o0, o1, o2, o3);
    const T c = (T)0.70710678118654752440084436210484903928;
    const T d = (T)DIR;
    const C2<T> w1 = mk(c * (o1.x - d * o1.y), c * (d * o1.x + o1.y));
    const C2<T> w2 = mul_i<DIR>(o2);
    const C2<T> w3 = mk(c * (-o3.x - d * o3.y), c * (d * o3.x - o3.y));
    u[0] = e0 + o0;
    u[4] = e0 - o0;
    u[1] = e1 + w1;
    u[5] = e1 - w1;
    u[2] = e2 + w2;
    u[6] = e2 - w2;
    u[3] = e3 + w3;
    u[7] = e3 - w3;
  }
};

// ---- radix-R DFTs of twiddled inputs: sum_r u[r] w^r W_R^(r q) with
// w = e^{DIR 2 pi i j / N} ------------------------------------------------------
// As log2 R levels of radix-2 butterflies (a + w b, a - w b) with the factor
// w = c + i s held as (c, s/c): b + i (s/c) b takes two fused multiply-adds,
// and a +- c times that four.  Radix 8 so takes 72 against the 80 instructions
// of the products followed by the untwiddled DFT, and four factors to load
// (w^4, w^2, w, w W8; those turned by i are the same numbers) against seven.
// Every output goes through two roundings per level, the first of them of the
// size of w b alone: the FP32 error of a transform of 64 to 8192 points is 0.96
// to 0.99 of that of the products (forming a - w b as 2 a - (a + w b), also six
// instructions, hands the sum's rounding on to the difference: 1.10 to 1.14).
template <class T>
__device__ __forceinline__ void bfly(C2<T>& a, C2<T>& b, C2<T> w) {
  const T x = fma(-w.y, b.y, b.x), y = fma(w.y, b.x, b.y);
  b = mk(fma(-w.x, x, a.x), fma(-w.x, y, a.y));
  a = mk(fma(w.x, x, a.x), fma(w.x, y, a.y));
}
// the same with the factor DIR i w
template <int DIR, class T>
__device__ __forceinline__ void bfly_i(C2<T>& a, C2<T>& b, C2<T> w) {
  const T x = fma(-w.y, b.y, b.x), y = fma(w.y, b.x, b.y), c = DIR * w.x;
  b = mk(fma(c, y, a.x), fma(-c, x, a.y));
  a = mk(fma(-c, y, a.x), fma(c, x, a.y));
}
template <int DIR, class T>
__device__ __forceinline__ C2<T> turn(C2<T> w) {  // tables hold the forward sign
  return DIR > 0 ? conj(w) : w;
}

// The factor table of length N: entry j < N/2 is e^{-2 pi i j / N} as (c, s/c),
// formed in long double, s/c with the rounded c so that s = c (s/c) carries one
// rounding (with the angle and its functions in FP64 the FP64 transforms' error
// is 1.2 to 1.5 times as large: 2.7e-16 against 1.8e-16 at 512 points).  A
// quarter turn has c = 0: 2^-30 (2^-60 in FP64) stands for it, at most 1/32 of
// the other factors' rounding; a quarter turn of values above 3e29 (1e290)
// overflows.
template <class T>
void fft_factors(int N, C2<T>* w) {
  for (int j = 0; j <= N / 4; ++j) {
    const long double a = 2 * 3.14159265358979323846264338327950288L * j / N;
    const T c = 4 * j == N ? std::ldexp((T)1, sizeof(T) == 8 ? -60 : -30) : (T)std::cos(a);
    w[j].x = c;
    w[j].y = (T)(-std::sin(a) / c);
    if (j > 0 && 4 * j < N) {  // e^{-i (pi - a)}
      w[N / 2 - j].x = -c;
      w[N / 2 - j].y = -w[j].y;
    }
  }
}

// The four factors a thread's butterflies of one stage take: those of its one
// radix-8 butterfly, of its two radix-4 or of its four radix-2 ones.
template <int N, int R, int P, class T>
__device__ __forceinline__ void load_factors(C2<T> (&w)[4], const C2<T>* __restrict__ tw, int t) {
  constexpr int TT = N / kFftE, NB = kFftE / R;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int j = ((t + b * TT) & (P - 1)) * (N / (P * R));
    if constexpr (R == 8) {
      w[0] = tw[4 * j];
      w[1] = tw[2 * j];
      w[2] = tw[j];
      w[3] = tw[j + N / 8];
    } else if constexpr (R == 4) {
      w[2 * b] = tw[2 * j];
      w[2 * b + 1] = tw[j];
    } else {
      w[b] = tw[j];
    }
  }
}

template <int R, int DIR, class T>
struct DftTw;  // run(u, factors, butterfly)

template <int DIR, class T>
struct DftTw<2, DIR, T> {
  __device__ static __forceinline__ void run(C2<T> (&u)[2], const C2<T> (&f)[4], int b) {
    bfly(u[0], u[1], turn<DIR>(f[b]));
  }
};

template <int DIR, class T>
struct DftTw<4, DIR, T> {
  __device__ static __forceinline__ void run(C2<T> (&u)[4], const C2<T> (&f)[4], int b) {
    const C2<T> w2 = turn<DIR>(f[2 * b]), w = turn<DIR>(f[2 * b + 1]);
    bfly(u[0], u[2], w2);  // even q, odd q
    bfly(u[1], u[3], w2);
    bfly(u[0], u[1], w);         // q = 0, 2
    bfly_i<DIR>(u[2], u[3], w);  // q = 1, 3
    const C2<T> x = u[1];
    u[1] = u[2];
    u[2] = x;
  }
};

template <int DIR, class T>
struct DftTw<8, DIR, T> {
  __device__ static __forceinline__ void run(C2<T> (&u)[8], const C2<T> (&f)[4], int) {
    const C2<T> w4 = turn<DIR>(f[0]), w2 = turn<DIR>(f[1]), w = turn<DIR>(f[2]), w1 = turn<DIR>(f[3]);
#pragma unroll
    for (int a = 0; a < 4; ++a) bfly(u[a], u[a + 4], w4);  // even q in 0..3, odd in 4..7
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      bfly(u[a], u[a + 2], w2);                // q mod 4 = 0, 2
      bfly_i<DIR>(u[4 + a], u[6 + a], w2);  // q mod 4 = 1, 3
    }
    bfly(u[0], u[1], w);          // q = 0, 4
    bfly_i<DIR>(u[2], u[3], w);   // q = 2, 6
    bfly(u[4], u[5], w1);         // q = 1, 5
    bfly_i<DIR>(u[6], u[7], w1);  // q = 3, 7
    const C2<T> x1 = u[1], x3 = u[3], x6 = u[6];
    u[1] = u[4];
    u[4] = x1;
    u[3] = x6;
    u[6] = x3;
  }
};

// Where the stages take their factors from: the table in memory, stage by
// stage, or registers filled beforehand (Factors), which takes the table's
// latency out of the transforms' serial chain.
template <class T>
struct Table {
  const C2<T>* __restrict__ tw;
  template <int N, int R, int P, int S>
  __device__ __forceinline__ void get(C2<T> (&w)[4], int t) const {
    load_factors<N, R, P>(w, tw, t);
  }
};
template <int N, class T, int SCH = kSchedDefault>
struct Factors {
  C2<T> f[3][4];  // twiddled stages of sizes up to 1024
  template <int P = 1, int S = 0>
  __device__ __forceinline__ void load(const C2<T>* __restrict__ tw, int t) {
    constexpr int R = stage_radix<N, SCH>(P);
    if constexpr (P > 1) {
      static_assert(S < 3, "stages");
      load_factors<N, R, P>(f[S], tw, t);
    }
    if constexpr (P * R < N) load<P * R, (P > 1 ? S + 1 : 0)>(tw, t);
  }
  template <int, int, int, int S>
  __device__ __forceinline__ void get(C2<T> (&w)[4], int) const {
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = f[S][q];
  }
};

// Orders the LDS accesses between the stages of a transform group.  With
// WAVE, the group's workgroup is a single wavefront: the LDS unit executes one
// wavefront's instructions in issue order, so a store is seen by every later
// load of the same wavefront, and a load is not overtaken by a later store,
// without a barrier or a wait for either to complete; a wavefront-scope fence
// (which emits no instruction) keeps the compiler from moving the one across
// the other.  Otherwise a workgroup barrier.
template <bool WAVE>
__device__ __forceinline__ void lds_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// ---- one Stockham stage, recursing into the next ---------------------------
// v[f][e] holds element t + e*TT of transform f.  `lds` points at this group's
// fft_slots(NF) regions of Padded<N> entries each.  tw: the table
// of fft_factors, or its entries of every stage (Factors).
template <int N, int DIR, int NF, int P, class T, int SCH, bool WAVE, int S = 0>
struct FftStage {
  static constexpr int E = kFftE;
  static constexpr int TT = N / E;
  static constexpr int R = stage_radix<N, SCH>(P);
  static_assert(R == 2 || R == 4 || R == 8, "radix");
  static constexpr int NB = E / R;  // butterflies per thread in this stage
  static constexpr bool LAST = (P * R == N);
  static constexpr int NP = Padded<N, SCH>::value;

  // twiddle multiplication and radix-R DFT of the NB butterflies of transform
  // f; the outputs go back to registers (last stage) or to LDS region `slot`
  __device__ static __forceinline__ void butterflies(C2<T> (&v)[NF][E], int f, C2<T>* slot, int t,
                                                     const C2<T> (&w)[4]) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int i = t + b * TT;
      const int k = i & (P - 1);
      C2<T> u[R];
#pragma unroll
      for (int r = 0; r < R; ++r) u[r] = v[f][b + r * NB];
      if constexpr (P > 1)
        DftTw<R, DIR, T>::run(u, w, b);
      else
        Dft<R, DIR, T>::run(u);
      if constexpr (LAST) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[f][b + r * NB] = u[r];
      } else {
        const int j0 = lds_pad<SCH>((i - k) * R + k);
#pragma unroll
        for (int r = 0; r < R; ++r) slot[j0 + lds_step<SCH>(r * P)] = u[r];
      }
    }
  }

  __device__ static __forceinline__ void gather(C2<T> (&v)[NF][E], int f, const C2<T>* slot, int t) {
    const int j0 = lds_pad<SCH>(t);
#pragma unroll
    for (int e = 0; e < E; ++e) v[f][e] = slot[j0 + lds_step<SCH>(e * TT)];
  }

  template <class F>
  __device__ static __forceinline__ void run(C2<T> (&v)[NF][E], C2<T>* lds, int t, const F& tw) {
    constexpr int NS = fft_slots(NF, WAVE);
    constexpr int SN = P > 1 ? S + 1 : 0;
    C2<T> w[4];
    if constexpr (P > 1) tw.template get<N, R, P, S>(w, t);
    if constexpr (LAST) {
#pragma unroll
      for (int f = 0; f < NF; ++f) butterflies(v, f, lds, t, w);
    } else if constexpr (NS == NF) {
#pragma unroll
      for (int f = 0; f < NF; ++f) butterflies(v, f, lds + f * NP, t, w);
      lds_sync<WAVE>();
#pragma unroll
      for (int f = 0; f < NF; ++f) gather(v, f, lds + f * NP, t);
      lds_sync<WAVE>();
      FftStage<N, DIR, NF, P * R, T, SCH, WAVE, SN>::run(v, lds, t, tw);
    } else {
      // transform f uses slot f % NS; with several slots the barrier after
      // writing f also orders every read of f - NS (issued before it) ahead of
      // the reuse of its slot, with one the reads of f - 1 need their own
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        if (NS == 1 && f > 0) lds_sync<WAVE>();
        butterflies(v, f, lds + (f % NS) * NP, t, w);
        lds_sync<WAVE>();
        gather(v, f, lds + (f % NS) * NP, t);
      }
      lds_sync<WAVE>();
      FftStage<N, DIR, NF, P * R, T, SCH, WAVE, SN>::run(v, lds, t, tw);
    }
  }
};

// Unnormalised transform(s): out[m] = sum_n in[n] e^{DIR 2 pi i m n / N}.
// WAVE: the calling workgroup is one wavefront (see lds_sync).
template <int N, int DIR, int NF, int SCH = kSchedDefault, bool WAVE = false, class T>
__device__ __forceinline__ void fft(C2<T> (&v)[NF][kFftE], C2<T>* lds, int t,
                                    const C2<T>* __restrict__ tw) {
  static_assert(N >= 64 && (N & (N - 1)) == 0, "N must be a power of two >= 64");
  FftStage<N, DIR, NF, 1, T, SCH, WAVE>::run(v, lds, t, Table<T>{tw});
}
// the same with the factors at hand
template <int N, int DIR, int NF, int SCH = kSchedDefault, bool WAVE = false, class T>
__device__ __forceinline__ void fft(C2<T> (&v)[NF][kFftE], C2<T>* lds, int t, const Factors<N, T, SCH>& tw) {
  FftStage<N, DIR, NF, 1, T, SCH, WAVE>::run(v, lds, t, tw);
}

}  // namespace ttsh
