"""Host-side checks of the fused kernels' plans (no GPU).

The sweep kernel covers a lattice with waves of 64 lanes x vec columns marching
down chunks of rows, each collided with 4 columns and rows more than it stores;
the tile kernel with tiles of its region shapes.  These tests build the plan
functions of the kernels' headers for the host (tests/host_plans.hip) and check
that every node is stored by one wave or tile, and that a sweep's stored columns
have the columns they depend on in the same wave, in order, across the seam of a
ragged periodic row.
"""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
STEPS = 4


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("plans") / "libhost_plans.so")
    subprocess.check_call([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1705_11092_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "host_plans.hip")])
    lib = ctypes.CDLL(out)
    lib.host_sweep_plan.restype = ctypes.c_double
    lib.host_tile_plan.restype = ctypes.c_double
    lib.host_tile_plan.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong, ctypes.c_int, ctypes.c_void_p]
    return lib


@pytest.mark.parametrize("max_vec", [1, 2])
@pytest.mark.parametrize("nx,ny", [(64, 64), (65, 1000), (112, 4096), (113, 70), (239, 3000), (240, 3000), (241, 64),
                                   (1024, 1024), (1501, 703), (4096, 4096), (4097, 2049), (16384, 64)])
def test_sweep_plan_stores_every_node_once(plans, nx, ny, max_vec):
    o = (ctypes.c_int * 6)()
    plans.host_sweep_plan(nx, ny, 4, 1024, max_vec, o)
    vec, strips, rows, units, groups, halo = o
    assert 1 <= vec <= max_vec and groups == -(-nx // vec)
    chunks = -(-ny // rows)
    assert units == strips * chunks and (chunks - 1) * rows < ny <= chunks * rows
    last = nx - (groups - 1) * vec  # real columns of the row's last group
    stored = [0] * nx
    for s in range(strips):
        lanes = []
        for lane in range(64):
            q = s * (64 - 2 * halo) + lane - halo
            g = q % groups
            real = list(range(g * vec, g * vec + (last if g == groups - 1 else vec)))
            lanes.append((real, halo <= lane < 64 - halo and q < groups))
        cols = [c for real, _ in lanes for c in real]
        assert all((b - a) % nx == 1 % nx for a, b in zip(cols, cols[1:]))
        at = 0
        for real, store in lanes:
            if store:
                # One column of a level's result is lost at each end per step.
                assert at >= STEPS and len(cols) - at - len(real) >= STEPS
                for c in real:
                    stored[c] += 1
            at += len(real)
    assert stored == [1] * nx


@pytest.mark.parametrize("storage", range(6))
@pytest.mark.parametrize("nx,ny", [(1, 1), (18, 10), (19, 11), (58, 26), (64, 32), (200, 200), (512, 512), (64, 4096),
                                   (1030, 9), (2048, 2048)])
def test_tile_plans_cover_the_lattice(plans, nx, ny, storage):
    o = (ctypes.c_int * 6)()
    eb = 8 if storage == 0 else (4 if storage == 1 else 2)
    us = plans.host_tile_plan(nx, ny, storage, 9 * nx * ny * eb, 256, o)
    steps, shape, tiles_x, tiles, tw, th = o
    assert us > 0 and steps in (4, 8) and 0 <= shape < 6 and tw >= 1 and th >= 1
    assert (tiles_x - 1) * tw < nx <= tiles_x * tw
    tiles_y = tiles // tiles_x
    assert tiles == tiles_x * tiles_y and (tiles_y - 1) * th < ny <= tiles_y * th
    plans.host_sc_tile_plan(nx, ny, storage, 256, o)
    steps, shape, tiles_x, tiles = o[:4]
    w, h = {4: (18, 10), 2: (58, 26)}[steps]
    assert shape == {4: 6, 2: 7}[steps]
    assert tiles_x == -(-nx // w) and tiles == tiles_x * -(-ny // h)
