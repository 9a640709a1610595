// host_plans.hip -- TEST INFRASTRUCTURE: the plans of the fused kernels
// (sweep_plan, tile_plan and their modelled times, from the kernels' headers)
// compiled for the host, so that a CPU test can check what they cover.  Built
// by tests/test_fused_cpu.py with hipcc --offload-host-only; never part of the
// library.
#include "clbm_internal.h"

extern "C" {
// out: vec, strips, rows, units, groups, halo.  Returns us per step.
double host_sweep_plan(int nx, int ny, int eb, int simds, int max_vec, int *out)
{
    const clbm::SweepPlan p = clbm::sweep_plan(nx, ny, eb, simds, max_vec);
    const int v[6] = {p.vec, p.strips, p.rows, p.units, p.groups, p.halo};
    for (int k = 0; k < 6; ++k) out[k] = v[k];
    return clbm::sweep_us((int64_t)nx * ny, eb, simds, p.vec, p.halo, p.rows, p.units) / clbm::kSweepSteps;
}

// out: steps, shape, tiles across, tiles, tile width, tile height.  Returns us
// per step.
double host_tile_plan(int nx, int ny, int storage, long long bytes, int cus, int *out)
{
    double us = 0.0;
    const clbm::TilePlan p = clbm::tile_plan(nx, ny, storage, bytes, cus, &us);
    const int v[6] = {p.steps, p.shape, p.tiles_x, p.tiles, clbm::region_tile_w(p.shape),
                      clbm::region_tile_h(p.shape)};
    for (int k = 0; k < 6; ++k) out[k] = v[k];
    return us;
}

void host_sc_tile_plan(int nx, int ny, int storage, int cus, int *out)
{
    const clbm::TilePlan p = clbm::sc_tile_plan(nx, ny, storage, cus);
    out[0] = p.steps;
    out[1] = p.shape;
    out[2] = p.tiles_x;
    out[3] = p.tiles;
}
}
