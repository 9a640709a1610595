"""Which kernel a run takes (Lattice.next_launch), and that each route gives the
one-step kernel's result bitwise.
"""
import pytest

pytestmark = pytest.mark.gpu

RATES = (1.0, 1.2, 1.25, 1.25, 1.1, 1.1)


def _lattice(nx, ny, storage, bc=0, force="const", inplace=False, scheme="consistent"):
    from paper_1705_11092_amd import inputs
    from tests.gpu_util import gpu_lattice
    wl = inputs.random_state(nx, ny, seed=nx + 3 * ny, bc_y=bc, force=force, amp_f=1e-4, amp_u=0.02, s=RATES)
    return gpu_lattice(wl, storage, scheme, inplace=inplace)


def test_bench_names_the_kernel_that_runs():
    import bench
    for storage, n, kernel in (("f16", 512, "k_tile"), ("f32", 512, "k_tile"), ("f32", 4096, "k_sweep")):
        bench.run_gpu(n, storage, 8, 0)
        assert bench.kernel_label(bench.run_gpu.launch).startswith(kernel + " (")
    bench.run_gpu(512, "f16", 8, 0, pairs=False)
    assert bench.kernel_label(bench.run_gpu.launch) == "k_step"
