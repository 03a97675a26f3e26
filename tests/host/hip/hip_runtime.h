// Stand-in for the HIP runtime header in host builds of device headers: one
// lane is one fiber, and every fence or barrier hands over to the next lane
// (lanes.hpp).
#pragma once
#include <cmath>
#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
void lane_yield();
inline void __syncthreads() { lane_yield(); }
// a macro, as the scope argument of the builtin is a string literal
#define __builtin_amdgcn_fence(order, scope) lane_yield()
using std::fma;
