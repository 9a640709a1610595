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


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_resident_kernel_follows_what_the_lattice_steps_with(storage):
    # Tiny lattices that step singly or in pairs run in the resident block;
    # those that step in LDS tiles do not, unless a limit asks for it.
    for pairs in (False, True):
        lat = _lattice(16, 16, storage)
        assert lat.next_launch(10)[:2] == ("tiles", 8)
        lat.step_pairs = pairs
        assert lat.next_launch(10)[:2] == ("resident", 10)
        assert lat.next_launch(1)[:2] == ("step", 1)
        lat.step_pairs = None
        assert lat.next_launch(10)[:2] == ("tiles", 8)
        lat.set_resident_limit(1 << 20)
        assert lat.next_launch(10)[:2] == ("resident", 10)
        lat.step_pairs = pairs
        lat.set_resident_limit(0)
        assert lat.next_launch(10)[0] == ("pair" if pairs else "step")
        lat.close()
    lat = _lattice(16, 16, storage, inplace=True)
    assert lat.next_launch(10)[:2] == ("resident", 10)
    lat.close()
    big = _lattice(100, 100, storage)
    big.step_pairs = False
    assert big.next_launch(10)[0] == "step"
    big.close()


@pytest.mark.parametrize("storage,nx,ny,bc,one,two", [
    ("f64", 40, 30, 1, "tiles", "tiles"),       # one round of tiles
    ("f64", 384, 380, 0, "step", "pair"),       # little work
    ("f64", 1024, 1000, 1, "tiles", "tiles"),   # in the Infinity Cache
    ("f64", 1450, 1460, 0, "step", "pair"),     # beyond it
    ("f32", 512, 500, 1, "step", "tiles"),
    ("f32", 1500, 1400, 0, "tiles", "tiles"),
    ("f32", 16, 20000, 0, "step", "tiles"),     # tiles cover more than the lattice
    ("f32", 64, 20003, 0, "step", "pair"),      # and more than the pairs' tiles
    ("f16", 768, 760, 0, "step", "tiles"),
    ("f16", 1500, 1490, 0, "tiles", "tiles"),
    ("f16sr", 1500, 1490, 1, "step", "pair"),   # 16-bit between walls
    ("bf16", 2800, 2750, 0, "step", "pair"),    # beyond the Infinity Cache
])
def test_last_steps_of_a_run_take_the_cheaper_kernel(storage, nx, ny, bc, one, two):
    import torch
    lat, ref = (_lattice(nx, ny, storage, bc) for _ in range(2))
    assert lat.next_launch(3)[0] == lat.next_launch(9)[0] == "tiles"
    assert lat.next_launch(1)[:2] == (one, 1)
    assert lat.next_launch(2)[:2] == (two, 2)
    ref.step_pairs = False
    ref.set_resident_limit(0)
    most = lat.next_launch(9)[1]
    for n in (1, 2, most + 1, most + 2):
        lat.step(n)
        ref.step(n)
    assert torch.equal(lat.get_populations(), ref.get_populations())
    lat.close()
    ref.close()


def test_16_bit_plans_weigh_walls_and_force_fields():
    # The tall regions lose a block per compute unit to walls and fields.
    import torch
    for storage, nx, ny, bc, force, want in [
            ("f16sr", 2900, 2890, 0, "const", ("tiles", 4, 64, 48)),
            ("f16sr", 2900, 2890, 0, "kolmogorov", ("tiles", 4, 64, 48)),
            ("f16sr", 2900, 2890, 0, "field", ("tiles", 4, 64, 32)),
            ("f16sr", 2900, 2890, 1, "const", ("pair", 2, 0, 0)),
            ("bf16", 2900, 2890, 1, "const", ("pair", 2, 0, 0)),
            ("f32", 1200, 1210, 1, "field", ("tiles", 4, 64, 32))]:
        lat, ref = (_lattice(nx, ny, storage, bc, force) for _ in range(2))
        assert lat.next_launch(8) == want, (storage, bc, force)
        ref.step_pairs = False
        lat.step(5)
        ref.step(5)
        assert torch.equal(lat.get_populations(), ref.get_populations()), (storage, bc, force)
        lat.close()
        ref.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16sr"])
def test_short_batch_calls_between_long_ones(storage):
    # Calls of one and two steps may step in pairs where longer ones step in
    # tiles; force changes in between regroup both.
    import torch

    from paper_1705_11092_amd import clbm
    sizes = [(700, 650), (640, 700), (333, 1000), (900, 400), (16, 16), (500, 777)]
    lats, refs = ([_lattice(nx, ny, storage, k % 2, ["const", "field", "kolmogorov"][k % 3])
                   for k, (nx, ny) in enumerate(sizes)] for _ in range(2))
    for lat in refs:
        lat.step_pairs = False
        lat.set_resident_limit(0)
    batch = clbm.Batch(lats)
    for call, n in enumerate((1, 9, 2, 1, 2, 5, 1, 70, 2, 3, 1)):
        counts = [n if (k + call) % 3 else n - 1 for k in range(len(lats))]
        batch.step_each(counts)
        for lat, c in zip(refs, counts):
            lat.step(c)
        if call in (3, 7):
            for lat in (lats[call % 6], refs[call % 6]):
                lat.set_force("kolmogorov", params=(2e-4, 2))
        for lat, ref, size in zip(lats, refs, sizes):
            assert torch.equal(lat.get_populations(), ref.get_populations()), (storage, call, size)
    batch.close()
    for lat in lats + refs:
        lat.close()


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_large_force_fields_and_populations_reach_every_node(storage):
    # More nodes than the force field's grid has threads.  Without momentum the
    # velocity is F / 2 rho; these forces (24 bits or fewer) are stored exactly.
    import torch

    from paper_1705_11092_amd import clbm
    nx, ny = 3100, 2803
    lat = clbm.Lattice(nx, ny, RATES, storage=storage)
    k = torch.arange(nx * ny, device="cuda", dtype=torch.float64).reshape(ny, nx)
    fx, fy = k * 2.0**-40, (nx * ny - k) * 2.0**-40
    lat.set_force("field", fx=fx, fy=fy)
    lat.set_populations(torch.ones((9, ny, nx), device="cuda", dtype=torch.float64))
    rho, ux, uy, _ = lat.moments(totals=False)
    assert torch.equal(ux, 0.5 * fx / rho) and torch.equal(uy, 0.5 * fy / rho)
    f = torch.rand((9, ny, nx), device="cuda", dtype=torch.float32).to(torch.float64)
    lat.set_populations(f)
    # The deviations from the rest weights are stored: one rounding each way.
    assert float((lat.get_populations() - f).abs().max()) <= (2.0**-52 if storage == "f64" else 2.0**-24)
    lat.close()
