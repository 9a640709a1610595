"""Graph replays, written slots and batch chunks of every step kernel, those that
lattices take by default among them (asserted).
"""
import pytest

from paper_1705_11092_amd import inputs
from tests.gpu_util import gpu_lattice

pytestmark = pytest.mark.gpu

RATES = (1.0, 1.2, 1.25, 1.25, 1.1, 1.1)


def _lattice(nx, ny, storage, bc=0, force="const", inplace=False):
    wl = inputs.random_state(nx, ny, seed=nx + 5 * ny, bc_y=bc, force=force, amp_f=1e-4, amp_u=0.02, s=RATES)
    return gpu_lattice(wl, storage, inplace=inplace)


@pytest.mark.parametrize("storage,nx,ny,pairs,inplace,graph,kind", [
    ("f64", 150, 90, None, False, 64, "tiles"),     # eight launches of eight steps
    ("f64", 150, 90, None, False, 72, "tiles"),     # nine: a replay flips the buffer
    ("f32", 700, 610, None, False, 36, "tiles"),    # nine of four
    ("f16sr", 600, 580, None, False, 38, "tiles"),  # and two steps more
    ("f32", 2060, 2100, None, False, 36, "sweep"),
    ("f32", 1024, 1000, True, False, -1, "pair"),   # by default
    ("f64", 300, 280, True, False, 66, "pair"),     # 33 launches
    ("f32", 1024, 1000, False, False, -1, "step"),
    ("f32", 1500, 900, False, True, -1, "step"),
    ("bf16", 300, 200, False, True, 64, "step"),
])
def test_graph_replays_match_direct_launches(storage, nx, ny, pairs, inplace, graph, kind):
    # Several replays with the program's own work and waits between them.
    import torch
    a, b = (_lattice(nx, ny, storage, 0 if inplace else 1, inplace=inplace) for _ in range(2))
    for lat in (a, b):
        lat.step_pairs = pairs
        lat.set_resident_limit(0)
    if graph >= 0:
        a.set_graph_steps(graph)
    b.set_graph_steps(0)
    assert a.next_launch(64)[0] == kind
    spare = torch.zeros(1 << 20, device="cuda")
    for n in (64, 1, 150, 72, 3, 36, 144, 66):
        a.step(n)
        b.step(n)
        spare.add_(1.0)
        if n % 2:
            torch.cuda.synchronize()
        assert torch.equal(a.get_populations(), b.get_populations()), n
    assert a.steps == b.steps
    a.close()
    b.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16", "f16sr", "bf16sr"])
@pytest.mark.parametrize("pairs,steps,kind", [(False, 1, "step"), (True, 2, "pair"), (None, 8, "tiles")])
def test_every_slot_written_by_each_kernel(storage, pairs, steps, kind):
    # NaN in the destination buffer before each launch: none may remain.
    import torch
    lat = _lattice(150, 37, storage, 1, "field")
    lat.step_pairs = pairs
    lat.set_resident_limit(0)
    assert lat.next_launch(steps)[:2] == (kind, steps)
    for k in range(3):
        (lat.pop_b if k % 2 == 0 else lat.pop_a).fill_(0xFF)
        lat.step(steps)
        assert bool(torch.isfinite(lat.get_populations()).all()), k
    lat.close()


@pytest.mark.parametrize("storage,nx,ny", [("f32", 2051, 2060), ("f64", 2051, 1900)])
def test_every_slot_written_by_sweeps(storage, nx, ny):
    import torch
    lat = _lattice(nx, ny, storage, 1, "field")
    assert lat.next_launch(4)[:2] == ("sweep", 4)
    for k in range(2):
        (lat.pop_b if k % 2 == 0 else lat.pop_a).fill_(0xFF)
        lat.step(4)
        assert bool(torch.isfinite(lat.get_populations()).all()), k
    lat.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16sr"])
def test_batches_of_tiles_and_in_place_lattices_through_several_chunks(storage):
    # In-place lattices step singly, so the batch replays graphs of 64 steps;
    # lattices in tiles go on through several of them, or end within one.
    import torch

    from paper_1705_11092_amd import clbm
    shapes = [(120, 70, 1, "field", False), (64, 33, 0, "const", True), (300, 250, 0, "const", False),
              (18, 10, 1, "const", False), (90, 90, 1, "kolmogorov", True), (33, 200, 0, "field", False)]
    lats, refs = ([_lattice(nx, ny, storage, bc, force, inplace) for nx, ny, bc, force, inplace in shapes]
                  for _ in range(2))
    batch = clbm.Batch(lats)
    for ref in refs:
        ref.step_pairs = False
        ref.set_resident_limit(0)
        ref.set_graph_steps(0)
    for counts in ([133, 200, 70, 65, 0, 64], [200, 3, 129, 127, 150, 191], [64, 64, 64, 64, 64, 64], [7, 140, 135, 1, 66, 2]):
        batch.step_each(counts)
        for ref, n in zip(refs, counts):
            ref.step(n)
        for lat, ref, shape in zip(lats, refs, shapes):
            assert lat.steps == ref.steps
            assert torch.equal(lat.get_populations(), ref.get_populations()), (shape, counts)
    batch.close()
    for lat in lats + refs:
        lat.close()


def test_captured_short_batch_calls():
    # Calls of one step have a plan of their own, whose tile map a captured call
    # must not leave to the replays: eager calls before a replay would read it.
    import torch

    from paper_1705_11092_amd import clbm
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        lats, refs = ([_lattice(nx, ny, "f16") for nx, ny in ((768, 760), (500, 700))] for _ in range(2))
        batch = clbm.Batch(lats, stream=stream)
        batch.step(9)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            batch.step(1)
            batch.step(1)  # two launches: the replay leaves each state in the buffer it took it from
        batch.step(1)      # eager, before any replay
        batch.step(1)
        for _ in range(3):
            graph.replay()
        batch.step(1)
        for ref in refs:
            ref.step_pairs = False
            ref.step(9 + 2 + 3 * 2 + 1)
        for lat, ref in zip(lats, refs):
            assert torch.equal(lat.get_populations(), ref.get_populations())
        batch.close()
        for lat in lats + refs:
            lat.close()
