// host_routes.hip -- TEST INFRASTRUCTURE: rules of clbm_internal.h that choose
// routes (graph_steps, tiles_take), compiled for the host.  Built by
// tests/test_routes_cpu.py with hipcc --offload-host-only; never part of the
// library.
#include "clbm_internal.h"

extern "C" {
int host_graph_steps(int asked, int fused, long long bytes) { return clbm::graph_steps(asked, fused, bytes); }
}
