// Real fields from a spectrum that lives on the 1/2-rule disk, and the
// projection of real fields onto it, in FP64 (read-out, diagnostics and the
// surrogate's coarse fields; not in the time loop).
//
// A field of the disk has M+1 = N/4+1 columns m_x >= 0 and, being real, needs
// no others: the column kernel transforms each stored column of each
// component along y, and the row kernel rebuilds the negative m_x by
// conjugation, transforms v_x + i v_y of a row at once and writes the result
// in its final form.  Between them lies G [M+1][N] (column, row) with the
// components of an entry side by side.
// The kernels are bound by latency at the common sizes (a 512^2 field is
// 2 MB of G): two launches in place of five or six full-size passes over a
// complex N x N array.
#pragma once

#include "fft.hpp"

namespace ttsh {

template <int N>
struct Readout {
  static constexpr int TT = N / kFftE;
  static constexpr int M = N / 4;
  static constexpr int NP = Padded<N>::value;
  // a wavefront per workgroup for the small sizes, and enough workgroups to
  // spread one field over the chip for the others
  static constexpr int CPB = N <= 256 ? 512 / N : N <= 1024 ? 2 : 1;                        // columns per workgroup
  static constexpr int RPB = N <= 128 ? 512 / N : N <= 1024 ? 4 : N == 2048 ? 2 : 1;  // rows per workgroup
  // the kernels' reductions exchange values between all 64 lanes of a wavefront
  static_assert(CPB * TT % 64 == 0 && RPB * TT % 64 == 0, "whole wavefronts");
  // LDS regions of a column's transforms: all of an 8192-point column's LDS
  // goes to one region
  static constexpr int SLOTS = N <= 4096 ? 2 : 1;
};

// the NC transforms of v, together if two regions fit, else one by one
template <int N, int DIR, int NC, bool WAVE>
__device__ __forceinline__ void fft_each(C2<double> (&v)[NC][kFftE], C2<double>* lds, int t,
                                         const C2<double>* __restrict__ tw) {
  if constexpr (NC == 1 || Readout<N>::SLOTS == 2) {
    fft<N, DIR, NC, kSchedDefault, WAVE>(v, lds, t, tw);
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      C2<double> w[1][kFftE];
#pragma unroll
      for (int e = 0; e < kFftE; ++e) w[0][e] = v[c][e];
      fft<N, DIR, 1, kSchedDefault, WAVE>(w, lds, t, tw);
#pragma unroll
      for (int e = 0; e < kFftE; ++e) v[c][e] = w[0][e];
    }
  }
}

// components of G: the velocity, the vorticity or both
enum { kCompV = 1, kCompW = 2, kCompVW = 3 };
constexpr int comp_count(int comp) { return (comp & kCompV ? 2 : 0) + (comp & kCompW ? 1 : 0); }

// columns 0..Mk of the state of an Ns grid, taken to an N grid by mode index
// (modes beyond either radius are zero), scaled to the values of the field
template <int N, class S, int COMP>
__global__ void __launch_bounds__(Readout<N>::CPB* Readout<N>::TT)
synth_cols(const C2<S>* __restrict__ st, int Ns, int Mk, double dk, C2<double>* __restrict__ G,
           const C2<double>* __restrict__ tw) {
  using R = Readout<N>;
  constexpr int NC = comp_count(COMP), NT = R::CPB * R::TT;
  constexpr int REG = NC == 1 ? 1 : R::SLOTS;
  __shared__ C2<double> lds[R::CPB * REG * R::NP];
  const int t = threadIdx.x % R::TT, col = threadIdx.x / R::TT;
  const int mx = blockIdx.x * R::CPB + col;
  const int MPs = Ns / 4 + 1, SPs = Ns / 2 + 2;
  const double s = 1.0 / Ns;
  C2<double> v[NC][kFftE];
#pragma unroll
  for (int e = 0; e < kFftE; ++e) {
    const int idx = t + e * R::TT;
    const int my = idx <= R::M ? idx : idx - N;
    C2<double> a = mk(0.0, 0.0), b = mk(0.0, 0.0);
    if ((idx <= R::M || idx >= N - R::M) && mx * mx + my * my <= Mk * Mk) {
      const int pos = my >= 0 ? my : my + SPs - 1;
      a = cscale(cvt<double>(st[mx * SPs + pos]), s);
      b = cscale(cvt<double>(st[(MPs + mx) * SPs + pos]), s);
    }
    if constexpr (COMP & kCompV) {
      v[0][e] = a;
      v[1][e] = b;
    }
    if constexpr (COMP & kCompW) {  // i dk (m_x v_y - m_y v_x)
      const C2<double> c = cscale(b, (double)mx) - cscale(a, (double)my);
      v[NC - 1][e] = mk(-c.y * dk, c.x * dk);
    }
  }
  fft_each<N, +1, NC, NT == 64>(v, lds + col * REG * R::NP, t, tw);
  if (mx <= Mk) {
#pragma unroll
    for (int e = 0; e < kFftE; ++e) {
      C2<double>* g = G + ((size_t)mx * N + t + e * R::TT) * NC;
#pragma unroll
      for (int c = 0; c < NC; ++c) g[c] = v[c][e];
    }
  }
}

// what a row of the field becomes
enum { kOutFloat = 0, kOutPlanar = 1, kOutComplex = 2, kOutReal = 3, kOutOrder = 4 };
struct RowsOut {
  const C2<double>* G;  // [batch][Mk+1][N][components]
  const C2<double>* tw;
  void* out;
  long long stride;  // kOutFloat: floats from one pixel to the next
  int batch;
  int Mk;
  int kind;
  int comp;
  int vec;  // kOutFloat: pixels are 8-byte aligned
  double dx, cx, cy, D;  // kOutOrder
};

// Per-workgroup partials of the order parameters (kOutOrder): sums of
// |v_theta| and |v|, and for the left and right region the largest |omega|
// with its node and signed value.
constexpr int kOrderPart = 8;

// The larger |omega| of two candidates; equal values go to the lower node.
__host__ __device__ __forceinline__ void order_best(double& a, double& i, double& w, double a2, double i2, double w2) {
  if (a2 > a || (a2 == a && a2 >= 0.0 && i2 < i)) {
    a = a2;
    i = i2;
    w = w2;
  }
}

template <int N, int OUT, int COMP>
__global__ void __launch_bounds__(Readout<N>::RPB* Readout<N>::TT) synth_rows(RowsOut a) {
  using R = Readout<N>;
  constexpr int NC = comp_count(COMP), NT = R::RPB * R::TT, BPI = N / R::RPB;
  constexpr int NZ = (COMP & kCompV ? 1 : 0) + (COMP & kCompW ? 1 : 0);
  __shared__ C2<double> lds[R::RPB * R::NP];
  const int tid = threadIdx.x, lane = tid % R::RPB, t = tid / R::RPB;
  const int b = blockIdx.x / BPI, y = (blockIdx.x - b * BPI) * R::RPB + lane;
  const C2<double>* G = a.G + (size_t)b * (a.Mk + 1) * N * NC;
  C2<double> z[NZ][kFftE];
#pragma unroll
  for (int e = 0; e < kFftE; ++e) {
    const int idx = t + e * R::TT;
    const bool hi = idx > N / 2;
    const int m = hi ? N - idx : idx;
#pragma unroll
    for (int q = 0; q < NZ; ++q) z[q][e] = mk(0.0, 0.0);
    if (m <= a.Mk) {
      const C2<double>* g = G + ((size_t)m * N + y) * NC;
      if constexpr (COMP & kCompV) {
        C2<double> p = g[0], q = g[1];
        if (hi) {
          p = conj(p);
          q = conj(q);
        }
        z[0][e] = mk(p.x - q.y, p.y + q.x);
      }
      if constexpr (COMP & kCompW) z[NZ - 1][e] = hi ? conj(g[NC - 1]) : g[NC - 1];
    }
  }
#pragma unroll
  for (int q = 0; q < NZ; ++q) {
    C2<double> w[1][kFftE];
#pragma unroll
    for (int e = 0; e < kFftE; ++e) w[0][e] = z[q][e];
    fft<N, +1, 1, kSchedDefault, NT == 64>(w, lds + lane * R::NP, t, a.tw);
#pragma unroll
    for (int e = 0; e < kFftE; ++e) z[q][e] = w[0][e];
  }
  const size_t row = (size_t)b * N * N + (size_t)y * N;
  if constexpr (OUT == kOutFloat) {
    float* o = (float*)a.out;
#pragma unroll
    for (int e = 0; e < kFftE; ++e) {
      float* p = o + (long long)(row + t + e * R::TT) * a.stride;
      if (a.vec) {
        *(float2*)p = make_float2((float)z[0][e].x, (float)z[0][e].y);
      } else {
        p[0] = (float)z[0][e].x;
        p[1] = (float)z[0][e].y;
      }
    }
  } else if constexpr (OUT == kOutPlanar) {
    double* o = (double*)a.out;
#pragma unroll
    for (int e = 0; e < kFftE; ++e) {
      o[row + t + e * R::TT] = z[0][e].x;
      o[(size_t)N * N + row + t + e * R::TT] = z[0][e].y;
    }
  } else if constexpr (OUT == kOutComplex) {
    C2<double>* o = (C2<double>*)a.out;
#pragma unroll
    for (int e = 0; e < kFftE; ++e) o[row + t + e * R::TT] = z[0][e];
  } else if constexpr (OUT == kOutReal) {
    double* o = (double*)a.out;
#pragma unroll
    for (int e = 0; e < kFftE; ++e) o[row + t + e * R::TT] = z[0][e].x;
  } else {
    double num = 0.0, den = 0.0, ba[2] = {-1.0, -1.0}, bi[2] = {0.0, 0.0}, bw[2] = {0.0, 0.0};
    // the disk test rounds every product and sum separately (no fused
    // multiply-add), so that a node on a disk's rim falls on the same side as
    // in a plain evaluation of the same expression
    const double r2 = __dmul_rn(0.5 * a.D, 0.5 * a.D);
    const double cl = __dsub_rn(a.cx, 0.5 * a.D), cr = __dadd_rn(a.cx, 0.5 * a.D);
    const double yn = __dmul_rn((double)(y - N / 2), a.dx);
#pragma unroll
    for (int e = 0; e < kFftE; ++e) {
      const int x = t + e * R::TT;
      if constexpr (COMP & kCompV) {
        const double px = (x - N / 2) * a.dx - a.cx, py = (y - N / 2) * a.dx - a.cy;
        const double r = sqrt(px * px + py * py);
        const C2<double> v = z[0][e];
        if (r > 0.0) num += fabs((-py * v.x + px * v.y) / r);
        den += sqrt(v.x * v.x + v.y * v.y);
      }
      const double xn = __dmul_rn((double)(x - N / 2), a.dx);
      const int side = xn < a.cx ? 0 : 1;
      bool in = true;
      if (a.D > 0.0) {
        const double ex = __dsub_rn(xn, side ? cr : cl), ey = __dsub_rn(yn, a.cy);
        in = !(__dadd_rn(__dmul_rn(ex, ex), __dmul_rn(ey, ey)) > r2);
      }
      const double w = z[NZ - 1][e].x;
      if (in) {
        if (side)
          order_best(ba[1], bi[1], bw[1], fabs(w), (double)(y * N + x), w);
        else
          order_best(ba[0], bi[0], bw[0], fabs(w), (double)(y * N + x), w);
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      num += __shfl_xor(num, o, 64);
      den += __shfl_xor(den, o, 64);
#pragma unroll
      for (int s = 0; s < 2; ++s)
        order_best(ba[s], bi[s], bw[s], __shfl_xor(ba[s], o, 64), __shfl_xor(bi[s], o, 64), __shfl_xor(bw[s], o, 64));
    }
    double* red = reinterpret_cast<double*>(lds);
    __syncthreads();
    if ((tid & 63) == 0) {
      double* p = red + (tid >> 6) * kOrderPart;
      p[0] = num;
      p[1] = den;
      for (int s = 0; s < 2; ++s) {
        p[2 + 3 * s] = ba[s];
        p[3 + 3 * s] = bi[s];
        p[4 + 3 * s] = bw[s];
      }
    }
    __syncthreads();
    if (tid == 0) {
      for (int w = 1; w < NT / 64; ++w) {
        const double* p = red + w * kOrderPart;
        num += p[0];
        den += p[1];
        for (int s = 0; s < 2; ++s) order_best(ba[s], bi[s], bw[s], p[2 + 3 * s], p[3 + 3 * s], p[4 + 3 * s]);
      }
      double* p = (double*)a.out + (size_t)blockIdx.x * kOrderPart;
      p[0] = num;
      p[1] = den;
      for (int s = 0; s < 2; ++s) {
        p[2 + 3 * s] = ba[s];
        p[3 + 3 * s] = bi[s];
        p[4 + 3 * s] = bw[s];
      }
    }
  }
}

// ---- projection of batched real fields onto the disk ----------------------------
// rows: float pixels (v_x, v_y) -> W = FFT(v_x + i v_y) of the row at m and
// N - m, m = 0..M, side by side in G [batch][M+1][N][2]; the column kernel,
// whose thread loads both, separates the components
template <int N>
__global__ void __launch_bounds__(Readout<N>::RPB* Readout<N>::TT)
project_rows(const float* __restrict__ v, long long stride, C2<double>* __restrict__ G,
             const C2<double>* __restrict__ tw) {
  using R = Readout<N>;
  constexpr int NT = R::RPB * R::TT, BPI = N / R::RPB;
  __shared__ C2<double> lds[R::RPB * R::NP];
  const int tid = threadIdx.x, lane = tid % R::RPB, t = tid / R::RPB;
  const int b = blockIdx.x / BPI, y = (blockIdx.x - b * BPI) * R::RPB + lane;
  const float* p = v + ((long long)b * N * N + (long long)y * N) * stride;
  C2<double> z[1][kFftE];
#pragma unroll
  for (int e = 0; e < kFftE; ++e) {
    const float* q = p + (long long)(t + e * R::TT) * stride;
    z[0][e] = mk((double)q[0], (double)q[1]);
  }
  fft<N, -1, 1, kSchedDefault, NT == 64>(z, lds + lane * R::NP, t, tw);
  C2<double>* g = G + ((size_t)b * (R::M + 1) * N + y) * 2;
#pragma unroll
  for (int e = 0; e < kFftE; ++e) {
    const int idx = t + e * R::TT, m = (N - idx) & (N - 1);
    if (idx <= R::M) g[(size_t)idx * N * 2] = z[0][e];
    if (m <= R::M) g[(size_t)m * N * 2 + 1] = z[0][e];
  }
}

// columns: forward transform, cutoff, divergence-free part, inverse transform
// back into G as the components synth_rows takes; with `part`, the
// workgroup's share of the sums |v|^2 and (m x v)^2 over the spectrum
// (columns m_x > 0 stand for two)
template <int N>
__global__ void __launch_bounds__(Readout<N>::CPB* Readout<N>::TT)
project_cols(C2<double>* __restrict__ G, double* __restrict__ part, const C2<double>* __restrict__ tw) {
  using R = Readout<N>;
  constexpr int NT = R::CPB * R::TT, REG = R::SLOTS, CB = R::M / R::CPB + 1;
  __shared__ C2<double> lds[R::CPB * REG * R::NP];
  const int t = threadIdx.x % R::TT, col = threadIdx.x / R::TT;
  const int b = blockIdx.x / CB, mx = (blockIdx.x - b * CB) * R::CPB + col;
  C2<double>* g = G + ((size_t)b * (R::M + 1) + mx) * N * 2;
  const bool valid = mx <= R::M;
  C2<double> v[2][kFftE];
#pragma unroll
  for (int e = 0; e < kFftE; ++e) {
    C2<double> p = mk(0.0, 0.0), q = p;
    if (valid) {
      p = g[(t + e * R::TT) * 2];
      q = g[(t + e * R::TT) * 2 + 1];
    }
    v[0][e] = cscale(mk(p.x + q.x, p.y - q.y), 0.5);
    v[1][e] = cscale(mk(p.y + q.y, -(p.x - q.x)), 0.5);
  }
  fft_each<N, -1, 2, NT == 64>(v, lds + col * REG * R::NP, t, tw);
  double sv = 0.0, sw = 0.0;
  const double s = 1.0 / ((double)N * N);
#pragma unroll
  for (int e = 0; e < kFftE; ++e) {
    const int idx = t + e * R::TT;
    const int my = idx <= R::M ? idx : idx - N, m2 = mx * mx + my * my;
    C2<double> x = mk(0.0, 0.0), y = x;
    if ((idx <= R::M || idx >= N - R::M) && m2 <= R::M * R::M) {
      x = v[0][e];
      y = v[1][e];
      if (m2 > 0) {
        const C2<double> d = cscale(mk(mx * x.x + my * y.x, mx * x.y + my * y.y), 1.0 / m2);
        x = x - cscale(d, (double)mx);
        y = y - cscale(d, (double)my);
      }
      const C2<double> c = cscale(y, (double)mx) - cscale(x, (double)my);
      sv += x.x * x.x + x.y * x.y + y.x * y.x + y.y * y.y;
      sw += c.x * c.x + c.y * c.y;
    }
    v[0][e] = cscale(x, s);
    v[1][e] = cscale(y, s);
  }
  fft_each<N, +1, 2, NT == 64>(v, lds + col * REG * R::NP, t, tw);
  if (valid) {
#pragma unroll
    for (int e = 0; e < kFftE; ++e) {
      g[(t + e * R::TT) * 2] = v[0][e];
      g[(t + e * R::TT) * 2 + 1] = v[1][e];
    }
  }
  if (part) {
    if (mx > 0) {
      sv *= 2.0;
      sw *= 2.0;
    }
    sv = wave_sum_from(sv, 1);
    sw = wave_sum_from(sw, 1);
    double* red = reinterpret_cast<double*>(lds);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
      red[(threadIdx.x >> 6) * 2] = sv;
      red[(threadIdx.x >> 6) * 2 + 1] = sw;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < NT / 64; ++w) {
        sv += red[2 * w];
        sw += red[2 * w + 1];
      }
      part[2 * (size_t)blockIdx.x] = sv * s;  // Parseval for the unnormalised transform
      part[2 * (size_t)blockIdx.x + 1] = sw * s;
    }
  }
}

}  // namespace ttsh
