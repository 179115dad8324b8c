// One CG iteration's vector work of a small problem in one launch.
#pragma once

#include <cstdint>

#include "kernels.hpp"

namespace ndmg {

// Between two V-cycles, per pair (z = B r given): r . z (and z . q), beta, the pending u +=
// alpha p, p = z + beta p, q = A p, p . q, alpha, r -= alpha q (and r in FP32), r . r: what
// launch_dot, launch_cg_direction, launch_apply, launch_dot and launch_cg_update do, with the
// scalars in the same slots; first: p = z (no beta, no pending update).  With one pair also
// launch_pcg_check's test (nact, hist); with more the test is a launch of its own, on rr_part
// with one partial per pair.
struct CgStep {
  double *r, *p, *q, *u;
  float* r32;                    // may be null
  double* scal;
  int *act, *iters, *status;
  double* hist;
  int* nact;                     // one pair: receives the count of active pairs
  double* rr_part;
  int64_t pstride;
  int i_num, i_den, i_zq, i_an;  // slots as launch_cg_direction takes them
  int flexible, first;
};
// meshes of 2 .. kCgStepMaxN elements per axis (at most 5 unknowns per lane), constant alpha
constexpr int kCgStepMaxN = 12;
template <typename TZ>
hipError_t launch_cg_step(const TZ* z, const CgStep& s, const Geom& g, const Bat& bt, hipStream_t st);

}  // namespace ndmg
