// Many time steps of small grids in one launch: one workgroup holds an
// instance's mixed-domain fields in LDS and its spectrum in registers from
// step to step, so that nothing crosses workgroups and a step costs six
// workgroup barriers instead of two kernel launches with cold caches.
//
// The arithmetic is that of row_body and col_body (MODE 0).  A workgroup has
// N/2 x N/8 threads: thread (p, t) carries row pair p in the row part and, for
// p <= N/4, column m_x = p in the column part, elements t + e N/8 of it.  A
// transform's N/8 threads lie within one wavefront, so its exchanges need no
// barrier.  One LDS region serves in turn as X [3][M+1][N], the row
// transforms' exchange, Y [2 or 3][M+1][N] and the columns' exchange.
//
// Bound by latency in the one compute unit that an instance has: at 64^2 a
// wavefront per SIMD (FP64: about a quarter of the unit's rate) takes 7.4 us a
// step (9.2 us in FP64) against 12.2 (14.1) for two launches with one instance;
// at 128^2 four per SIMD take 19 to 21 us for up to 256 instances, 23 to 28 with
// the vorticity source, against 38 and 43 us for 256 (FP32; where the lines
// cross: resident_rule.hpp).
#pragma once

#include "step_multi.hpp"

namespace ttsh {

struct ResidentArgs {
  ClassArgs c;
  double beta, gamma_v, lambda0, gamma_w;
  LinCoef lc;
  int steps;
};

template <int N, class T, bool GW>
struct Resident {
  using G = Geo<N>;
  static constexpr int TT = G::TT, MP = G::MP, NT = N / 2 * TT, NC = MP * TT;
  // rows of the region: two rows' values of a column are one 16- (32-) byte
  // access, consecutive columns four banks apart
  static constexpr int LP = N + 16 / (int)sizeof(C2<T>);
  static constexpr int PS = (G::NP + 31) / 32 * 32 + 8;  // exchange entries per transform group
  static constexpr size_t xy = (size_t)3 * MP * LP * sizeof(C2<T>), ex = (size_t)N / 2 * PS * sizeof(C2<T>);
  static constexpr size_t region = ((xy > ex ? xy : ex) + 15) / 16 * 16;
  static constexpr int KEPT = 5;  // elements of a column that can hold kept modes
  static constexpr size_t tables = (size_t)2 * KEPT * NC * sizeof(double);
  static constexpr size_t herm = (size_t)N * sizeof(C2<double>);
  // 1024 threads leave 128 registers each: the column's state stays in memory
  // (the L2) and the factors in LDS instead of being held in registers
  static constexpr bool TIGHT = NT > 512;
  static constexpr size_t factors = TIGHT ? N / 2 * sizeof(C2<T>) : 0;
  static constexpr size_t bytes = region + tables + herm + factors + (NT / 64) * 2 * sizeof(double);
};

// the transforms' factors: registers, or the table in LDS
template <int N, class T, bool TIGHT>
struct ResidentFactors {
  Factors<N, T> f;
  __device__ __forceinline__ void init(const C2<T>* tw, C2<T>*, int t, int) { f.load(tw, t); }
  template <int DIR, int NF>
  __device__ __forceinline__ void run(C2<T> (&v)[NF][kFftE], C2<T>* lds, int t) const {
    fft<N, DIR, NF, kSchedDefault, true>(v, lds, t, f);
  }
};
template <int N, class T>
struct ResidentFactors<N, T, true> {
  const C2<T>* f;
  __device__ __forceinline__ void init(const C2<T>* tw, C2<T>* lds, int, int tid) {
    if (tid < N / 2) lds[tid] = tw[tid];
    f = lds;
  }
  template <int DIR, int NF>
  __device__ __forceinline__ void run(C2<T> (&v)[NF][kFftE], C2<T>* lds, int t) const {
    fft<N, DIR, NF, kSchedDefault, true>(v, lds, t, f);
  }
};

// sum over the TT consecutive lanes of a transform group
template <int TT, class T>
__device__ __forceinline__ T group_sum(T v) {
#pragma unroll
  for (int o = 1; o < TT; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <int N, class T, class S, bool GW>
__global__ void __launch_bounds__(N* N / 16) steps_resident(ResidentArgs a) {
  using R = Resident<N, T, GW>;
  using G = Geo<N>;
  constexpr int E = G::E, TT = G::TT, M = G::M, MP = G::MP, SP = G::SP, LP = R::LP, NFY = GW ? 3 : 2;
  extern __shared__ __align__(16) unsigned char smem[];
  C2<T>* reg = reinterpret_cast<C2<T>*>(smem);
  double* tabA = reinterpret_cast<double*>(smem + R::region);
  double* tabB = tabA + R::KEPT * R::NC;
  C2<double>* H = reinterpret_cast<C2<double>*>(smem + R::region + R::tables);
  C2<T>* twl = reinterpret_cast<C2<T>*>(smem + R::region + R::tables + R::herm);
  double* red = reinterpret_cast<double*>(smem + R::region + R::tables + R::herm + R::factors);

  const int tid = threadIdx.x;
  int p = tid / TT, t = tid % TT;
  __builtin_assume(t >= 0 && t < TT);
  const size_t inst = blockIdx.x;
  const ClassArgs& d = a.c;
  const bool valid = p <= M;                     // this thread has a column
  const bool busy = (tid & ~63) < R::NC;         // its wavefront has one
  int y0 = 2 * p, mx = p;
  C2<T>* L = reg + p * R::PS;
  ResidentFactors<N, T, R::TIGHT> fac;
  fac.init((const C2<T>*)d.tw, twl, t, tid);
  const T beta = (T)a.beta, gamma_v = (T)a.gamma_v, lambda0 = (T)a.lambda0, gamma_w = (T)a.gamma_w;
  const double dk = d.dk[inst], dt_over_N = a.lc.dt / N, sN = 1.0 / N;
  const T* Kp = (const T*)d.K + inst * N * N;
  C2<T>* Xg = (C2<T>*)d.X_out + inst * 3 * G::MP4 * N;
  C2<S>* stp = (C2<S>*)d.st + inst * 2 * MP * SP;

  // element e of a column: its m_y, kept or not, and its slot in the tables
  auto kept = [&](int e) {
    const int idx = t + e * TT;
    const int my = idx <= M ? idx : idx - N;
    return (idx <= M || idx >= N - M) && mx * mx + my * my <= M * M && valid;
  };
  auto my_of = [&](int e) { return t + e * TT <= M ? t + e * TT : t + e * TT - N; };
  auto pos_of = [&](int e) { return t + e * TT <= M ? t + e * TT : t + e * TT - (N - 2 * M - 1); };
  constexpr int slot_e[R::KEPT] = {0, 1, 2, E - 2, E - 1};

  // the column's part of the state, its linear factors, and X
  C2<S> sx[R::KEPT], sy[R::KEPT];
  auto load_state = [&] {
#pragma unroll
    for (int q = 0; q < R::KEPT; ++q) {
      const int e = slot_e[q];
      sx[q] = sy[q] = mk<S>(0, 0);
      if (kept(e)) {
        sx[q] = stp[mx * SP + pos_of(e)];
        sy[q] = stp[(MP + mx) * SP + pos_of(e)];
      }
    }
  };
  auto store_state = [&] {
#pragma unroll
    for (int q = 0; q < R::KEPT; ++q) {
      const int e = slot_e[q];
      if (kept(e)) {
        stp[mx * SP + pos_of(e)] = sx[q];
        stp[(MP + mx) * SP + pos_of(e)] = sy[q];
      }
    }
  };
  if (busy) {
    if constexpr (!R::TIGHT) load_state();
#pragma unroll
    for (int q = 0; q < R::KEPT; ++q) {
      const int e = slot_e[q];
      if (kept(e)) {
        double A, B;
        linear_ab<0>(a.lc, dk, mx * mx + my_of(e) * my_of(e), A, B);
        tabA[q * R::NC + tid] = A;
        tabB[q * R::NC + tid] = B * dt_over_N;
      }
    }
    if (valid) {
#pragma unroll
      for (int f = 0; f < 3; ++f)
#pragma unroll
        for (int e = 0; e < E; ++e) reg[(f * MP + mx) * LP + t + e * TT] = Xg[mix_idx<N>(f, mx, t + e * TT)];
    }
  }
  __syncthreads();

  for (int step = 0; step < a.steps; ++step) {
    // opaque, so that the mask, the modes' constants and the addresses are
    // formed in each step instead of being kept in (and spilled from)
    // registers through all of them
    asm volatile("" : "+v"(t), "+v"(p));
    __builtin_assume(t >= 0 && t < TT);
    y0 = 2 * p;
    mx = p;
    L = reg + p * R::PS;
    // ---- rows: X -> forcing -> Y ----
    C2<T> z[3][E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int idx = t + e * TT;
      const bool lo = idx <= M, hi = idx >= N - M;
      const int m = lo ? idx : N - idx;
      CPair<T> u, v, w;
      u.a = u.b = v.a = v.b = w.a = w.b = mk<T>(0, 0);
      if (lo || hi) {
        const C2<T>* q = reg + m * LP + y0;
        u.a = q[0];
        u.b = q[1];
        v.a = q[MP * LP];
        v.b = q[MP * LP + 1];
        w.a = q[2 * MP * LP];
        w.b = q[2 * MP * LP + 1];
      }
      if (idx == 0) u.a.y = u.b.y = v.a.y = v.b.y = w.a.y = w.b.y = 0;
      if (hi) {
        u.a = conj(u.a); u.b = conj(u.b);
        v.a = conj(v.a); v.b = conj(v.b);
        w.a = conj(w.a); w.b = conj(w.b);
      }
      z[0][e] = pack_pq(u.a, v.a);
      z[1][e] = pack_pq(u.b, v.b);
      z[2][e] = pack_pq(w.a, w.b);
    }
    __syncthreads();
    fac.template run<+1, 3>(z, L, t);
    T kr[2][E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      kr[0][e] = Kp[y0 * N + t + e * TT];
      kr[1][e] = Kp[(y0 + 1) * N + t + e * TT];
    }
    C2<T> wv[NFY][E];
    T s1[2][2] = {{0, 0}, {0, 0}};
#pragma unroll
    for (int e = 0; e < E; ++e) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const T vx = z[r][e].x, vy = z[r][e].y;
        const T om = r ? z[2][e].y : z[2][e].x;
        const T s = beta * (vx * vx + vy * vy) + gamma_v * kr[r][e];
        const T r1x = -s * vx, r1y = -s * vy;
        s1[r][0] += r1x;
        s1[r][1] += r1y;
        wv[r][e] = mk(r1x + lambda0 * om * vy, r1y - lambda0 * om * vx);
      }
      if constexpr (GW) wv[NFY - 1][e] = mk(-gamma_w * kr[0][e] * z[2][e].x, -gamma_w * kr[1][e] * z[2][e].y);
    }
    fac.template run<-1, NFY>(wv, L, t);
    {  // row sums, then their sum over the wavefront's rows
      double b[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        b[c] = (double)group_sum<TT>(s1[0][c]) + (double)group_sum<TT>(s1[1][c]);
        b[c] = wave_sum_from(b[c], TT);
      }
      if ((tid & 63) == 0) {
        red[2 * (tid >> 6)] = b[0];
        red[2 * (tid >> 6) + 1] = b[1];
      }
    }
    CPair<T> g[3];
    if constexpr (GW) {  // split the two rows' vorticity source
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int idx = t + e * TT;
        if (idx <= M || idx >= N - M) L[lds_pad(idx)] = wv[2][e];
      }
      lds_sync<true>();
      const T h = (T)0.5;
#pragma unroll
      for (int e = 0; e <= M / TT; ++e) {
        const int m = t + e * TT;
        if (m <= M) {
          const C2<T> Wm = L[lds_pad(m)], Wn = L[lds_pad((N - m) & (N - 1))];
          g[e].a = mk(h * (Wm.x + Wn.x), h * (Wm.y - Wn.y));
          g[e].b = mk(h * (Wm.y + Wn.y), -h * (Wm.x - Wn.x));
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int idx = t + e * TT, m = (N - idx) & (N - 1);
      if (idx <= M) {
        reg[idx * LP + y0] = wv[0][e];
        reg[idx * LP + y0 + 1] = wv[1][e];
      }
      if (m <= M) {
        reg[(MP + m) * LP + y0] = wv[0][e];
        reg[(MP + m) * LP + y0 + 1] = wv[1][e];
      }
      if constexpr (GW) {
        if (e <= M / TT && idx <= M) {
          reg[(2 * MP + idx) * LP + y0] = g[e < 3 ? e : 0].a;
          reg[(2 * MP + idx) * LP + y0 + 1] = g[e < 3 ? e : 0].b;
        }
      }
    }
    __syncthreads();

    // ---- columns: Y -> k-space update -> X ----
    C2<T> f[NFY][E], x[3][E];
    double s1x = 0.0, s1y = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) x[0][e] = x[1][e] = x[2][e] = mk<T>(0, 0);
    if (busy) {
      const T h = (T)0.5;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        C2<T> w0 = mk<T>(0, 0), w1 = w0, w2 = w0;
        if (valid) {
          const C2<T>* q = reg + mx * LP + t + e * TT;
          w0 = q[0];
          w1 = q[MP * LP];
          if constexpr (GW) w2 = q[2 * MP * LP];
        }
        f[0][e] = mk(h * (w0.x + w1.x), h * (w0.y - w1.y));
        f[1][e] = mk(h * (w0.y + w1.y), -h * (w0.x - w1.x));
        if constexpr (GW) f[2][e] = w2;
      }
#pragma unroll
      for (int w = 0; w < R::NT / 64; ++w) {
        s1x += red[2 * w];
        s1y += red[2 * w + 1];
      }
    }
    __syncthreads();
    if (busy) {
      fac.template run<-1, NFY>(f, L, t);
      C2<double> nx[R::KEPT], ny[R::KEPT];
#pragma unroll
      for (int q = 0; q < R::KEPT; ++q) {
        const int e = slot_e[q];
        nx[q] = ny[q] = mk(0.0, 0.0);
        if (kept(e)) {
          const int my = my_of(e), m2 = mx * mx + my * my;
          if constexpr (R::TIGHT) {
            sx[q] = stp[mx * SP + pos_of(e)];
            sy[q] = stp[(MP + mx) * SP + pos_of(e)];
          }
          const C2<double> ux = cvt<double>(sx[q]), uy = cvt<double>(sy[q]);
          const double A = tabA[q * R::NC + tid], bs = tabB[q * R::NC + tid];
          if (m2 == 0) {
            nx[q] = cscale(ux, A) + mk(bs * s1x, 0.0);
            ny[q] = cscale(uy, A) + mk(bs * s1y, 0.0);
          } else {
            double inv_m2;
            {  // as in col_body
              const double dm = (double)m2;
              double r = (double)__frcp_rn((float)m2);
              r = r * (2.0 - dm * r);
              inv_m2 = r * (2.0 - dm * r);
            }
            C2<double> qx = cscale(ux, A) + cscale(cvt<double>(f[0][e]), bs);
            C2<double> qy = cscale(uy, A) + cscale(cvt<double>(f[1][e]), bs);
            const double dmx = mx, dmy = my;
            const C2<double> dd = cscale(mk(dmx * qx.x + dmy * qy.x, dmx * qx.y + dmy * qy.y), inv_m2);
            qx = qx - cscale(dd, dmx);
            qy = qy - cscale(dd, dmy);
            if constexpr (GW) {
              const C2<double> gg = cscale(cvt<double>(f[NFY - 1][e]), bs * inv_m2 / dk);
              qx = qx + mk(-dmy * gg.y, dmy * gg.x);
              qy = qy + mk(dmx * gg.y, -dmx * gg.x);
            }
            nx[q] = qx;
            ny[q] = qy;
          }
        }
      }
      if ((tid >> 6) == 0) {  // Hermitian correction of the m_x = 0 column (lanes 0..TT-1), x then y
        auto fix = [&](C2<double>(&u)[R::KEPT]) {
          if (p == 0) {
#pragma unroll
            for (int q = 0; q < R::KEPT; ++q)
              if (kept(slot_e[q])) H[t + slot_e[q] * TT] = u[q];
          }
          lds_sync<true>();
          if (p == 0) {
#pragma unroll
            for (int q = 0; q < R::KEPT; ++q)
              if (kept(slot_e[q])) u[q] = cscale(u[q] + conj(H[(N - (t + slot_e[q] * TT)) & (N - 1)]), 0.5);
          }
          lds_sync<true>();
        };
        fix(nx);
        fix(ny);
      }
#pragma unroll
      for (int q = 0; q < R::KEPT; ++q) {
        const int e = slot_e[q];
        sx[q] = cvt<S>(nx[q]);
        sy[q] = cvt<S>(ny[q]);
        const C2<double> ux = cvt<double>(sx[q]), uy = cvt<double>(sy[q]);
        const double dmy = my_of(e);
        const C2<double> cw = cscale(uy, (double)mx) - cscale(ux, dmy);
        x[0][e] = cvt<T>(cscale(ux, sN));
        x[1][e] = cvt<T>(cscale(uy, sN));
        x[2][e] = cvt<T>(mk(-cw.y * dk * sN, cw.x * dk * sN));
      }
      if constexpr (R::TIGHT) store_state();
      fac.template run<+1, 3>(x, L, t);
    }
    __syncthreads();
    if (valid) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int e = 0; e < E; ++e) reg[(q * MP + mx) * LP + t + e * TT] = x[q][e];
    }
    __syncthreads();
  }

  if (valid) {
    if constexpr (!R::TIGHT) store_state();
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int e = 0; e < E; ++e) Xg[mix_idx<N>(f, mx, t + e * TT)] = reg[(f * MP + mx) * LP + t + e * TT];
  }
}

}  // namespace ttsh
