// Host-side launch interface between the runtime (ttsh_capi.hip) and the
// kernels compiled once per grid size (kernels_n.hip built with -DTTSH_N=...).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace ttsh {

struct MultiArgs;
struct RowsOut;

// Transforms outside the time loop, compiled per grid size.
struct SizeOps {
  // unnormalised 2D transform of `batch` N x N complex arrays in place;
  // dir = -1 forward, +1 inverse; fp64 selects double (else float) data
  hipError_t (*fft2)(void* a, int batch, int dir, int fp64, const void* tw, hipStream_t);
  // fields from spectra and the projection of fields (readout.hpp); tw: the
  // FP64 factors of this size
  hipError_t (*synth_cols)(const void* st, int st_fp64, int Ns, int Mk, double dk, int comp, void* G, const void* tw,
                           hipStream_t);
  hipError_t (*synth_rows)(const RowsOut&, hipStream_t);
  hipError_t (*project_rows)(const float* v, long long stride, int batch, void* G, const void* tw, hipStream_t);
  hipError_t (*project_cols)(void* G, int batch, double* part, const void* tw, hipStream_t);
  int row_groups;  // workgroups of synth_rows per field
  int col_groups;  // workgroups of project_cols per field
};

// Time-step passes over every size class of a context, compiled per
// arithmetic and workgroup size.  row is null for the FP64-state arithmetic
// (its row pass is the FP32 one).
struct MultiOps {
  hipError_t (*row)(const MultiArgs&, int gw, hipStream_t);
  hipError_t (*col)(const MultiArgs&, int gw, int mode, hipStream_t);
  // the same passes as one launch per size class
  hipError_t (*row_split)(const MultiArgs&, int gw, hipStream_t);
  hipError_t (*col_split)(const MultiArgs&, int gw, int mode, hipStream_t);
};

// The FP32 row pass and one-stage column pass with a non-default transform
// schedule, one launch over every size class (autotuner candidates).
struct SchedOps {
  hipError_t (*row)(const MultiArgs&, int gw, hipStream_t);
  hipError_t (*col)(const MultiArgs&, int gw, hipStream_t);
};
// schedules compiled besides the default, in the order the autotuner tries them
constexpr int kNumSchedVariants = 5;
constexpr int kSchedVariants[kNumSchedVariants] = {6, 10, 9, 7, 11};  // 2 PAD + SMALL_FIRST
const SchedOps* sched_ops(int bs, int sch);  // null for the default schedule or an unknown one

// The passes of one size class of the paper's production sizes (4096, 8192),
// whose workgroups have N/8 threads: `o` holds that class alone (c[0]).
struct BigOps {
  hipError_t (*row)(const MultiArgs& o, int gw, hipStream_t);
  hipError_t (*col)(const MultiArgs& o, int gw, int mode, hipStream_t);
};
constexpr int kMaxBlockN = 2048;  // the largest size served by the 64..256-thread kernels
const BigOps* big_ops(int N, int prec);  // null where the tiles do not fit (8192 in FP64)

// `steps` one-stage time steps of class q of m in one launch, for the sizes
// whose fields one workgroup holds (step_resident.hpp); hipErrorInvalidValue
// for the others.
hipError_t resident_32(const MultiArgs& m, int q, int gw, int steps, hipStream_t);
hipError_t resident_64(const MultiArgs& m, int q, int gw, int steps, hipStream_t);
hipError_t resident_96(const MultiArgs& m, int q, int gw, int steps, hipStream_t);

const SizeOps* size_ops(int N);
// record `msg` as the calling thread's last error (ttsh_last_error) and return code
int record_error(int code, const char* msg);
const MultiOps* multi_ops(int prec, int bs);

}  // namespace ttsh
