"""The fused multi-step kernels against the one-step kernel, bitwise.

By default a two-buffer lattice takes four or eight steps per launch: in LDS
tiles (small and medium lattices, and any with the Shan-Chen force), or marching
down the rows with four time levels in registers (large FP32 and FP64 ones).
Every node update is the one-step kernel's on the same values, so populations
are compared for equality: tile and strip edges, lattices smaller than a region,
walls, ragged rows, every force mode and storage type, and step counts that
leave every remainder.  The one-step kernel is held against the oracle
elsewhere.
"""
import pytest

from paper_1705_11092_amd import inputs
from tests.gpu_util import gpu_lattice, log

pytestmark = pytest.mark.gpu

RATES = (1.0, 1.2, 1.25, 1.25, 1.1, 1.1)
STORAGES = ["f64", "f32", "f16", "bf16", "f16sr", "bf16sr"]


def _final(wl, storage, scheme, fused, counts):
    lat = gpu_lattice(wl, storage, scheme)
    if not fused:
        lat.step_pairs = False
        lat.set_resident_limit(0)
    per = lat.steps_per_launch
    for n in counts:
        lat.step(n)
    f = lat.get_populations()
    lat.close()
    return f, per


def _same(wl, storage, scheme, counts):
    import torch
    a, per = _final(wl, storage, scheme, True, counts)
    b, one = _final(wl, storage, scheme, False, counts)
    assert one == 1
    assert bool(torch.isfinite(a).all())
    assert torch.equal(a, b), f"{wl.nx}x{wl.ny} bc={wl.bc_y} {wl.force_kind} {storage} {scheme} {counts}"
    return per


# Region tiles are 18 x 10, 18 x 18, 58 x 10, 26 x 10 and 58 x 26 nodes (58 x 42
# in large 16-bit lattices).
TILE_SHAPES = [(1, 1, 0, "const"), (3, 2, 1, "field"), (18, 10, 1, "kolmogorov"), (19, 11, 0, "field"),
               (17, 9, 1, "const"), (58, 26, 0, "kolmogorov"), (59, 27, 1, "field"), (57, 25, 1, "none"),
               (116, 52, 1, "field"), (117, 53, 0, "const"), (300, 130, 0, "field"), (257, 255, 1, "kolmogorov"),
               (385, 383, 1, "field"), (600, 500, 0, "kolmogorov"), (64, 1500, 1, "field"), (800, 811, 1, "const")]


@pytest.mark.parametrize("scheme", ["consistent", "guo_lbl"])
@pytest.mark.parametrize("storage", STORAGES)
def test_lds_tiles_match_one_step(storage, scheme):
    seen = set()
    for k, (nx, ny, bc, force) in enumerate(TILE_SHAPES):
        wl = inputs.random_state(nx, ny, seed=700 + k, bc_y=bc, force=force, amp_f=1e-4, amp_u=0.02, s=RATES)
        seen.add(_same(wl, storage, scheme, (1, 2, 3, 4, 7, 8, 13, 1 + k % 8)))
    log(f"lds tiles {storage} {scheme}: steps per launch {sorted(seen)}")
    assert {4, 8} <= seen


@pytest.mark.parametrize("storage", ["f16", "bf16", "f16sr", "bf16sr"])
def test_tall_16_bit_tiles_match_one_step(storage):
    # 58 x 42 tiles: full ones, a remainder of one column and row, one less.
    for nx, ny, bc, force in [(1566, 1554, 1, "field"), (1509, 1513, 0, "kolmogorov"), (1565, 1553, 1, "const")]:
        wl = inputs.random_state(nx, ny, seed=nx, bc_y=bc, force=force, amp_f=1e-4, amp_u=0.02, s=RATES)
        assert _same(wl, storage, "consistent", (4, 3)) == 4


@pytest.mark.parametrize("storage,nx,ny,bc,force,scheme", [
    ("f32", 2051, 1900, 0, "field", "consistent"),      # one column per lane
    ("f32", 2048, 2050, 1, "kolmogorov", "guo_lbl"),
    ("f32", 3001, 2999, 0, "const", "consistent"),      # two, with the seam of an odd row
    ("f32", 3003, 3000, 1, "field", "premnath"),
    ("f64", 2049, 2051, 1, "field", "guo_lbl"),
    ("f64", 3001, 2900, 0, "kolmogorov", "consistent"),
    ("f64", 64, 20003, 1, "const", "consistent"),       # the narrowest
])
def test_sweeps_match_one_step(storage, nx, ny, bc, force, scheme):
    wl = inputs.random_state(nx, ny, seed=nx, bc_y=bc, force=force, amp_f=1e-4, amp_u=0.02, s=RATES)
    assert _same(wl, storage, scheme, (4, 7)) == 4


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16sr"])
def test_shan_chen_tiles_match_the_psi_pass(storage):
    for k, (wl, scheme) in enumerate([
            (inputs.slab(n=9, width=4, ny=3), "consistent"), (inputs.droplet(n=18, R=5.0), "consistent"),
            (inputs.slab(n=67, width=30, ny=29), "consistent"), (inputs.droplet(n=59, R=14.0, scheme="guo_lbl"), "guo_lbl"),
            (inputs.droplet(n=333, R=60.0, s3=1.8), "consistent")]):
        assert _same(wl, storage, scheme, (1, 2, 3, 4, 9)) in (2, 4)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16sr"])
def test_batched_tiles_with_uneven_counts_match_one_step(storage):
    # Lattices with and without walls in one group, counts that end in every
    # remainder of a launch, a small batch (eight steps per launch) and one
    # whose tiles outnumber the compute units.
    import torch

    from paper_1705_11092_amd import clbm
    for sizes in ([(16, 16), (33, 9), (80, 41), (18, 10), (5, 7)], [(200, 190), (301, 257), (120, 333), (64, 64)] * 2):
        wls = [inputs.random_state(nx, ny, seed=800 + k, bc_y=k % 2, force=["const", "field", "kolmogorov"][k % 3],
                                   amp_f=1e-4, amp_u=0.02, s=RATES) for k, (nx, ny) in enumerate(sizes)]
        lats = [gpu_lattice(wl, storage) for wl in wls]
        batch = clbm.Batch(lats)
        totals = [0] * len(lats)
        for call in range(3):
            counts = [(5 * j + 17 * call) % 23 + 64 * (call == 2) for j in range(len(lats))]
            batch.step_each(counts)
            totals = [t + c for t, c in zip(totals, counts)]
        batch.step(9)
        for wl, lat, n in zip(wls, lats, totals):
            ref, _ = _final(wl, storage, "consistent", False, (n + 9,))
            assert torch.equal(lat.get_populations(), ref), f"{wl.nx}x{wl.ny} {storage}"
        batch.close()
        for lat in lats:
            lat.close()
