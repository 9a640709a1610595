// clbm_tile_f16.hip -- the multi-step LDS tile kernel for F16 storage.
#include "clbm_tile.h"

namespace clbm {
template hipError_t launch_tile_st<ST_F16>(const LatDesc &, int, int, const TilePlan &, hipStream_t);
}  // namespace clbm
