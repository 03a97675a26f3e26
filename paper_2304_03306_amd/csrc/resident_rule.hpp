// Which contexts step in resident workgroups (step_resident.hpp).
#pragma once

#include <algorithm>

namespace ttsh {

// n64 and n128 instances of 64 and 128 points (128: FP32 transforms), with or
// without the vorticity source, one-stage schemes.
//
// 64 points: always (FP32: a step takes 7.4 us for 1 to 256 instances against
// 12.2 to 17.5 with the two passes, 17.6 against 39.6 for 1024; FP64 9.1 to 9.8
// against 14.1 to 26.9, 36.4 against 68.1; with the source 43.3 against 80.5).
// 128 points: a workgroup fills a compute unit, so the instances go in rounds
// of 256 and a round costs the same for 100 instances as for 256, while the
// two passes' time grows with their number.  Microseconds of a step, resident
// against the passes:
//                     96         256        257        512        768         1024
//   no source   18.8/20.7  21.1/37.8  37.0/38.9  40.2/58.3  58.8/81.4  77.8/122.6
//   source      22.7/23.7  28.1/43.1  48.1/44.2  53.1/67.1  79.4/94.6  105.6/138.4
// The FP64 state adds 0 to 4 % to either.  With the source the last round
// therefore has to hold some before it pays (the passes tuned with two groups
// are 5 to 15 % faster than the table's, which the numbers allow for); beyond
// 1024 instances the passes' arrays have left the caches.
// Both sizes: the classes run one after the other, 7.4 us (9 with the source)
// that the passes, which take all sizes at once, do not pay: 1 + 96 instances
// 25.9/22.9 and 31.1/26.7, 1 + 128 25.8/28.4 and 33.3/32.8, 1 + 160 26.5/31.1 and
// 34.9/35.8, 128 + 96 26.0/28.7 and 31.3/33.1.
inline bool resident_pays(int n64, int n128, bool source) {
  if (n128 == 0) return true;
  if (n128 < 96) return false;
  const int rounds = (n128 + 255) / 256, last = n128 - 256 * (rounds - 1);
  if (rounds > 4) return true;
  constexpr int least[2][4] = {{96, 0, 0, 0}, {96, 128, 192, 96}};
  int need = least[source][rounds - 1];
  if (n64 > 0) need = std::max(need, source ? 168 : 128);
  return last + n64 / 2 >= need;
}

}  // namespace ttsh
