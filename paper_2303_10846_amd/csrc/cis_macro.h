// The coloured PR-SGS sweeps of the macroscopic systems as one dataflow launch (kernels in cis_macro.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cis_internal.h"

namespace cis {

// 64-bit words per cell in the exchange buffer: one 128-byte line, whose 16-byte chunk c ^ (cell & 7) holds double c
// of the increment as two tagged words (the swizzle spreads the chunks of neighbouring cells over the LDS banks).
constexpr int kFlowWords = 16;
constexpr int kFlowColors = 16;  // most non-empty colours of a dataflow launch

// The non-empty colours of a mesh and the wavefronts that own them: colour k's cells off[k] .. off[k] + n[k] - 1
// belong to wavefronts wave0[k] .. wave0[k + 1] - 1 (64 / lanes-per-cell cells each).
struct FlowPlan {
  int m = 0;           // non-empty colours; 0: no dataflow launch for this mesh
  bool local = false;  // the whole mesh in one workgroup of kFlowLocal threads, increments in LDS; else one
                       // workgroup of 64 threads per wavefront
  int32_t off[kFlowColors], n[kFlowColors], wave0[kFlowColors + 1];
};
constexpr int kFlowLocal = 1024;

// Dataflow state of one cis_state: the plan, the exchange buffer [nc][kFlowWords] (device) and the tag of the
// last version published in it.
struct Flow {
  FlowPlan plan;
  uint64_t* words = nullptr;
  uint32_t tag = 0;
};

// The plan for a mesh on the current device: m = 0 where the mesh has more than kFlowColors colours or more
// wavefronts than the dataflow launch takes.
FlowPlan flow_plan(const Dev& d, const int64_t* color_off, int64_t n_colors);

// Bit of Work::flag[0] set when a wait of a dataflow launch ran out (its results are then not valid).
constexpr int32_t kFlowStuck = 8;

// Step 4 in one launch (spectral radii, right-hand side, n_macro forward + backward sweep pairs and the
// predicted equilibrium); f.plan.m > 0.
hipError_t launch_macro_flow(const Dev& d, const Bufs& b, const Work& w, Flow& f, int n_macro, hipStream_t st);

// Mac^T u = t of the adjoint's block preconditioner, n_pairs sweep pairs from u = 0; f.plan.m > 0.  flag: as
// Work::flag.
hipError_t launch_adj_macro_flow(const Dev& d, const Bufs& b, Flow& f, const double* t, double* u, int n_pairs,
                                 int32_t* flag, hipStream_t st);

}  // namespace cis
