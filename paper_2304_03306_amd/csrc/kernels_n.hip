// The transforms outside the time loop for one grid size, TTSH_N (defined on
// the compiler command line: 64 to 8192): full arrays for the set-up paths,
// and the read-out and projection kernels.
#include "fft_full.hpp"
#include "launch.hpp"
#include "readout.hpp"

#ifndef TTSH_N
#error "define TTSH_N"
#endif

namespace ttsh {
namespace {

constexpr int N = TTSH_N;
constexpr int TT = N / kFftE;
template <class T, int DIR>
hipError_t fft2_t(void* p, int batch, const void* tw, hipStream_t s) {
  C2<T>* a = (C2<T>*)p;
  constexpr int RPB = FullFft<N>::RPB, CPB = FullFft<N>::CPB;
  const int rows = batch * N;
  hipLaunchKernelGGL((fft_rows<N, DIR, T>), dim3((rows + RPB - 1) / RPB), dim3(RPB * TT), 0, s, a,
                     rows, (const C2<T>*)tw);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((fft_cols<N, DIR, T>), dim3((rows + CPB - 1) / CPB), dim3(CPB * TT), 0, s, a,
                     rows, (const C2<T>*)tw);
  return hipGetLastError();
}

hipError_t fft2(void* a, int batch, int dir, int fp64, const void* tw, hipStream_t s) {
  if (fp64) return dir < 0 ? fft2_t<double, -1>(a, batch, tw, s) : fft2_t<double, +1>(a, batch, tw, s);
  return dir < 0 ? fft2_t<float, -1>(a, batch, tw, s) : fft2_t<float, +1>(a, batch, tw, s);
}

template <class S, int COMP>
void synth_cols_t(const void* st, int Ns, int Mk, double dk, void* G, const void* tw, hipStream_t s) {
  using R = Readout<N>;
  hipLaunchKernelGGL((synth_cols<N, S, COMP>), dim3(Mk / R::CPB + 1), dim3(R::CPB * R::TT), 0, s, (const C2<S>*)st, Ns,
                     Mk, dk, (C2<double>*)G, (const C2<double>*)tw);
}

hipError_t cols(const void* st, int st_fp64, int Ns, int Mk, double dk, int comp, void* G, const void* tw,
                hipStream_t s) {
  if (Mk < 0 || Mk > N / 4 || Mk > Ns / 4) return hipErrorInvalidValue;
  switch (comp * 2 + (st_fp64 ? 1 : 0)) {
    case 2 * kCompV: synth_cols_t<float, kCompV>(st, Ns, Mk, dk, G, tw, s); break;
    case 2 * kCompV + 1: synth_cols_t<double, kCompV>(st, Ns, Mk, dk, G, tw, s); break;
    case 2 * kCompW: synth_cols_t<float, kCompW>(st, Ns, Mk, dk, G, tw, s); break;
    case 2 * kCompW + 1: synth_cols_t<double, kCompW>(st, Ns, Mk, dk, G, tw, s); break;
    case 2 * kCompVW: synth_cols_t<float, kCompVW>(st, Ns, Mk, dk, G, tw, s); break;
    case 2 * kCompVW + 1: synth_cols_t<double, kCompVW>(st, Ns, Mk, dk, G, tw, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int OUT, int COMP>
void synth_rows_t(const RowsOut& a, hipStream_t s) {
  using R = Readout<N>;
  hipLaunchKernelGGL((synth_rows<N, OUT, COMP>), dim3((unsigned)(a.batch * (N / R::RPB))), dim3(R::RPB * R::TT), 0, s,
                     a);
}

hipError_t rows(const RowsOut& a, hipStream_t s) {
  switch (a.kind * 4 + a.comp) {
    case kOutFloat * 4 + kCompV: synth_rows_t<kOutFloat, kCompV>(a, s); break;
    case kOutPlanar * 4 + kCompV: synth_rows_t<kOutPlanar, kCompV>(a, s); break;
    case kOutComplex * 4 + kCompV: synth_rows_t<kOutComplex, kCompV>(a, s); break;
    case kOutReal * 4 + kCompW: synth_rows_t<kOutReal, kCompW>(a, s); break;
    case kOutOrder * 4 + kCompW: synth_rows_t<kOutOrder, kCompW>(a, s); break;
    case kOutOrder * 4 + kCompVW: synth_rows_t<kOutOrder, kCompVW>(a, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t proj_rows(const float* v, long long stride, int batch, void* G, const void* tw, hipStream_t s) {
  using R = Readout<N>;
  hipLaunchKernelGGL((project_rows<N>), dim3((unsigned)(batch * (N / R::RPB))), dim3(R::RPB * R::TT), 0, s, v, stride,
                     (C2<double>*)G, (const C2<double>*)tw);
  return hipGetLastError();
}

hipError_t proj_cols(void* G, int batch, double* part, const void* tw, hipStream_t s) {
  using R = Readout<N>;
  hipLaunchKernelGGL((project_cols<N>), dim3((unsigned)(batch * (R::M / R::CPB + 1))), dim3(R::CPB * R::TT), 0, s,
                     (C2<double>*)G, part, (const C2<double>*)tw);
  return hipGetLastError();
}

}  // namespace

#define TTSH_CAT2(a, b) a##b
#define TTSH_CAT(a, b) TTSH_CAT2(a, b)
const SizeOps* TTSH_CAT(ops_, TTSH_N)() {
  static const SizeOps ops = {fft2,      cols,
                              rows,      proj_rows,
                              proj_cols, N / Readout<N>::RPB,
                              Readout<N>::M / Readout<N>::CPB + 1};
  return &ops;
}

}  // namespace ttsh
