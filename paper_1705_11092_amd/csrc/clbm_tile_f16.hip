// clbm_tile_f16.hip -- the multi-step LDS tile kernels for F16 storage.
#include "clbm_tile.h"

namespace clbm {
template hipError_t launch_tile_st<ST_F16>(const LatDesc &, int, int, const TilePlan &, hipStream_t);
template hipError_t launch_batch_tile_st<ST_F16>(const LatDesc *, const int32_t *, int64_t, int, bool, int, int,
                                              hipStream_t);
}  // namespace clbm
