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
