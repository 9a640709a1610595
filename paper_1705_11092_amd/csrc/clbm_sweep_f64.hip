// clbm_sweep_f64.hip -- the four-step kernel for F64 storage.
#include "clbm_sweep.h"

namespace clbm {
template hipError_t launch_sweep_st<ST_F64>(const LatDesc &, int, const SweepPlan &, hipStream_t);
}  // namespace clbm
