"""Host-side checks of the rules that choose a run's route (no GPU): built from
the kernels' headers for the host (tests/host_routes.hip).
"""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("routes") / "libhost_routes.so")
    subprocess.check_call([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1705_11092_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "host_routes.hip")])
    lib = ctypes.CDLL(out)
    lib.host_graph_steps.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    lib.host_tiles_take.argtypes = [ctypes.c_longlong] + [ctypes.c_int] * 6
    return lib


def test_graph_steps(routes):
    g = routes.host_graph_steps
    mb = 1 << 20
    # Single steps and pairs: 64 by default up to 256 MB of traffic per step
    # (FP32 2000 x 1200, 1900^2, FP16 2600^2), and what is asked for.
    for nx, ny, eb in [(16, 16, 8), (800, 800, 8), (2000, 1200, 4), (1900, 1900, 4), (2600, 2600, 2)]:
        assert g(-1, 0, 9 * nx * ny * eb) == 64
    assert g(-1, 0, 128 * mb) == 64 and g(-1, 0, 128 * mb + 1) == 0
    for asked in (0, 2, 64, 4096):
        assert g(asked, 0, mb) == g(asked, 0, 1024 * mb) == asked
    # Fused launches: directly by default; a replay holds at least eight.
    for fused in (2, 4, 8):
        assert g(-1, fused, mb) == g(0, fused, mb) == 0
        assert g(8 * fused - 2, fused, mb) == g(2, fused, mb) == 0
        assert g(8 * fused, fused, mb) == 8 * fused
        assert g(4096, fused, mb) == 4096


def test_short_runs(routes):
    # tiles_take(left, region shape, storage, walls, nx, ny): what the last one or
    # two steps of a run take on 256 compute units; three and more are the tile
    # kernel's, and so is anything in one round of tiles.
    def take(left, shape, storage, walls, nx, ny):
        return bool(routes.host_tiles_take(left, shape, storage, walls, nx, ny, 256))
    R32X24, R32X32, R64X16, R32X16, R64X32, R64X48 = range(6)
    F64, F32, F16, BF16, F16_SR, BF16_SR = range(6)
    for storage in range(6):
        assert take(3, R64X32, storage, 1, 4096, 4096) and take(1, R32X24, storage, 1, 200, 180)
        # Beyond the Infinity Cache neither.
        assert not take(1, R64X32, storage, 0, 4096, 4096) and not take(2, R64X32, storage, 0, 4096, 4096)
    for shape, storage, walls, nx, ny, one, two in [
            (R64X16, F64, 0, 512, 512, False, False), (R64X16, F64, 1, 1024, 1024, True, True),
            (R32X16, F64, 0, 16, 20000, False, True), (R64X32, F32, 1, 1500, 1500, True, True),
            (R32X32, F32, 0, 16, 20000, False, True), (R32X16, F32, 0, 64, 20003, False, False),
            (R64X32, F16, 0, 1500, 1500, True, True), (R64X32, F16, 1, 1500, 1500, False, False),
            (R32X16, F16, 0, 32, 32768, False, False), (R64X48, BF16_SR, 0, 2048, 2048, True, True),
            (R64X16, BF16, 0, 768, 768, False, True)]:
        assert (take(1, shape, storage, walls, nx, ny), take(2, shape, storage, walls, nx, ny)) == (one, two)
