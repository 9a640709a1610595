// clbm_tile_f32.hip -- the multi-step LDS tile kernel for F32 storage.
#include "clbm_tile.h"

namespace clbm {
template hipError_t launch_tile_st<ST_F32>(const LatDesc &, int, int, const TilePlan &, hipStream_t);
}  // namespace clbm
