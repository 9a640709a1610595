// clbm_sweep_f32.hip -- the four-step kernel for F32 storage.
#include "clbm_sweep.h"

namespace clbm {
template hipError_t launch_sweep_st<ST_F32>(const LatDesc &, int, const SweepPlan &, hipStream_t);
}  // namespace clbm
