"""Every region shape of the tile kernels in every storage type, alone and in a
batch, against the one-step kernel, bitwise.

Sizes whose plan is the shape (asserted), with ragged tiles at the right and lower
edge; periodic with a constant force, and between walls with a force field.  A
batch of the same lattice takes the same plan.
"""
import pytest

from paper_1705_11092_amd import inputs
from tests.gpu_util import gpu_lattice

pytestmark = pytest.mark.gpu

RATES = (1.0, 1.2, 1.25, 1.25, 1.1, 1.1)
# (width, height of the region) -> steps of a launch
STEPS = {(32, 24): 8, (32, 32): 8, (64, 16): 4, (32, 16): 4, (64, 32): 4, (64, 48): 4}
PERIODIC = {
    "f64": {(32, 24): (37, 23), (32, 32): (10, 3000), (64, 16): (108, 1031), (32, 16): (24, 1296), (64, 32): (183, 1614)},
    "f32": {(32, 24): (37, 23), (32, 32): (10, 3000), (64, 16): (108, 1031), (32, 16): (1561, 38), (64, 32): (183, 1296)},
    "f16": {(32, 24): (37, 23), (32, 32): (10, 3000), (64, 16): (108, 1031), (32, 16): (1561, 38), (64, 32): (289, 1296),
            (64, 48): (1349, 1667)},
    "f16sr": {(32, 24): (37, 23), (32, 32): (10, 3000), (64, 16): (108, 1031), (32, 16): (24, 1296),
              (64, 32): (183, 1614), (64, 48): (1349, 1667)},
}
WALLED = {
    "f64": PERIODIC["f64"], "f32": PERIODIC["f32"],
    "f16": {(32, 24): (37, 23), (32, 32): (10, 3000), (64, 16): (289, 872), (32, 16): (1561, 38), (64, 32): (660, 1084),
            (64, 48): (766, 3000)},
    "f16sr": {(32, 24): (37, 23), (32, 32): (10, 3000), (64, 16): (108, 1031), (32, 16): (24, 1296),
              (64, 32): (289, 1296), (64, 48): (1667, 1455)},
}
LIKE = {"bf16": "f16", "bf16sr": "f16sr"}


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16", "f16sr", "bf16sr"])
@pytest.mark.parametrize("bc,force,scheme", [(0, "const", "guo_lbl"), (1, "field", "consistent")])
def test_every_region_matches_one_step(storage, bc, force, scheme):
    import torch

    from paper_1705_11092_amd import clbm
    sizes = (WALLED if bc else PERIODIC)[LIKE.get(storage, storage)]
    assert set(sizes) == {r for r in STEPS if r != (64, 48) or storage not in ("f64", "f32")}
    for region, (nx, ny) in sizes.items():
        k = STEPS[region]
        wl = inputs.random_state(nx, ny, seed=nx + ny, bc_y=bc, force=force, amp_f=1e-4, amp_u=0.02, s=RATES)
        lat, member, ref = (gpu_lattice(wl, storage, scheme) for _ in range(3))
        assert lat.next_launch(100) == ("tiles", k, *region)
        batch = clbm.Batch([member])
        ref.step_pairs = False
        ref.set_resident_limit(0)
        for n in (k, 2 * k + 3, 3):
            batch.step(n)
            for one in (lat, ref):
                one.step(n)
            f = ref.get_populations()
            assert torch.equal(lat.get_populations(), f), (region, nx, ny, n)
            assert torch.equal(member.get_populations(), f), (region, nx, ny, n, "batch")
        assert bool(torch.isfinite(f).all())
        batch.close()
        for one in (lat, member, ref):
            one.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16sr"])
@pytest.mark.parametrize("scheme", ["consistent", "guo_lbl"])
def test_both_shan_chen_regions_match_the_psi_pass(storage, scheme):
    # 32 x 24 regions of four steps and 64 x 32 of two, with remainders.
    import torch
    for n, region, k in ((450, (64, 32), 2), (512, (64, 32), 2), (333, (32, 24), 4), (700, (64, 32), 2)):
        wl = inputs.droplet(n=n, R=n / 6.0, s3=1.8, scheme=scheme)
        lat, ref = (gpu_lattice(wl, storage, scheme) for _ in range(2))
        assert lat.next_launch(100) == ("tiles", k, *region)
        ref.step_pairs = False
        assert ref.next_launch(100)[0] == "step"
        for steps in (1, k, 2 * k + 1, 3):
            lat.step(steps)
            ref.step(steps)
        f = lat.get_populations()
        assert bool(torch.isfinite(f).all())
        assert torch.equal(f, ref.get_populations()), (n, storage, scheme)
        lat.close()
        ref.close()
