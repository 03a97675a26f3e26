// Launchers of the resident time stepping (step_resident.hpp) for one
// arithmetic, TTSH_PREC = 32, 64 or 96 (set on the compiler command line): the
// grid sizes whose fields fit one workgroup's LDS (64 points per side, and 128
// with FP32 transforms).
#include "launch.hpp"
#include "step_resident.hpp"

#if !defined(TTSH_PREC)
#error "define TTSH_PREC"
#endif

namespace ttsh {
namespace {

#if TTSH_PREC == 64
using T = double;
using S = double;
#elif TTSH_PREC == 96
using T = float;
using S = double;
#else
using T = float;
using S = float;
#endif

template <int N, bool GW>
hipError_t go(const ResidentArgs& a, hipStream_t s) {
  using R = Resident<N, T, GW>;
  static_assert(R::bytes <= kMaxTileLds, "the fields must fit the LDS");
  hipLaunchKernelGGL((steps_resident<N, T, S, GW>), dim3(a.c.n), dim3(R::NT), R::bytes, s, a);
  return hipGetLastError();
}

hipError_t launch(const MultiArgs& m, int q, int gw, int steps, hipStream_t s) {
  const ResidentArgs a{m.c[q], m.beta, m.gamma_v, m.lambda0, m.gamma_w, m.lc, steps};
  switch (a.c.N) {
    case 64: return gw ? go<64, true>(a, s) : go<64, false>(a, s);
#if TTSH_PREC != 64
    case 128: return gw ? go<128, true>(a, s) : go<128, false>(a, s);
#endif
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

#define TTSH_CAT2(a, b) a##b
#define TTSH_CAT(a, b) TTSH_CAT2(a, b)
hipError_t TTSH_CAT(resident_, TTSH_PREC)(const MultiArgs& m, int q, int gw, int steps, hipStream_t s) {
  return launch(m, q, gw, steps, s);
}

}  // namespace ttsh
