// host_routes.hip -- TEST INFRASTRUCTURE: rules of clbm_internal.h that choose
// routes (graph_steps, tiles_take), compiled for the host.  Built by
// tests/test_routes_cpu.py with hipcc --offload-host-only; never part of the
// library.
#include "clbm_internal.h"

extern "C" {
int host_tiles_take(long long left, int shape, int storage, int walls, int nx, int ny, int cus)
{
    auto count = [&](int w, int h) { return (int64_t)((nx + w - 1) / w) * ((ny + h - 1) / h); };
    const int eb = storage == clbm::ST_F64 ? 8 : (storage == clbm::ST_F32 ? 4 : 2);
    const clbm::ShortRun r{shape, storage, walls != 0, count(clbm::region_tile_w(shape), clbm::region_tile_h(shape)),
                           count(clbm::tile_w(0), clbm::tile_h(0, storage)), (int64_t)nx * ny,
                           9 * clbm::row_pitch(nx, eb) * ny * eb};
    return clbm::tiles_take(left, r, cus);
}
int host_graph_steps(int asked, int fused, long long bytes) { return clbm::graph_steps(asked, fused, bytes); }
}
