"""Every form a batch is advanced in against single lattices stepped one by one:
the persistent grids of the single step's tiles, pairs of strips (directly and
from the captured graph), flat lattices.  Bit for bit: the tolerance is zero."""
import json

import pytest
import torch

from paper_1402_5487_amd import inputs
from paper_1402_5487_amd.batch import Batch
from paper_1402_5487_amd.lattice import Lattice

pytestmark = pytest.mark.gpu


def _start(sizes, tune=None, graph_steps=8):
    specs = [(nx, ny, 1.5 + 0.3 * i / len(sizes)) for i, (nx, ny) in enumerate(sizes)]
    b = Batch(specs)
    if tune is not None:
        b.autotune(tune)
    b.set_graph_steps(graph_steps)
    picks = sorted({0, len(sizes) - 1, *range(0, len(sizes), max(1, len(sizes) // 5))})
    lats = {}
    for i, (nx, ny, om) in enumerate(specs):
        fields = inputs.random_fields(nx, ny, seed=i)
        b.init(i, *fields)
        if i in picks:
            lats[i] = Lattice(2, nx, ny, omega=om, storage="f32").init(*fields)
    return b, lats


def _advance(b, lats, plan):
    for n in plan:
        b.step(n)
        for lat in lats.values():
            for _ in range(n):
                lat.step(1)
        for i, lat in lats.items():
            assert torch.equal(b.buffer(i), lat.f), (n, i, lat.nx, lat.ny)


@pytest.mark.parametrize("mode", [2, 4])
@pytest.mark.parametrize("w,r", [(64, 2), (256, 1)])
@pytest.mark.parametrize("listed", [False, True])
def test_persistent_grids_of_single_steps(mode, w, r, listed, tmp_path):
    """Calls of one step take the single step's tiles, more of them than the
    grid has workgroups, from either buffer; more than 48 sizes take the list."""
    sizes = [(100 + 2 * i, 90 + i % 7) for i in range(50)] * 4 if listed else [
        (64, 64), (100, 70), (130, 130), (256, 200), (7, 5), (1024, 1024), (512, 512), (320, 288), (480, 96)] * 2
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    entries = [{"arch": arch, "storage": "f32", "class": c, "w": w, "r": r} for c in sorted({max(s) for s in sizes})]
    path = tmp_path / "t.json"
    path.write_text(json.dumps({"entries": entries, "grid": {"arch": arch, "mode": mode, "lds": 40 * 1024}}))
    b, lats = _start(sizes, tune=path)
    info = b.info()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert info["grid_mode"] == mode and info["tiles"] > 2 * mode * cus
    _advance(b, lats, (1, 1, 1))
    b.close()


# 300 lattices of 70 x 70 take pairs of strips; 52 sizes beside them the list
@pytest.mark.parametrize("sizes", [[(70, 70)] * 300, [(70, 70)] * 300 + [(60 + i, 70) for i in range(52)]])
@pytest.mark.parametrize("graph_steps", [0, 2, 6, 8])
def test_pairs_of_strips(sizes, graph_steps):
    """Directly and from the graph, which starts from either buffer."""
    b, lats = _start(sizes, graph_steps=graph_steps)
    _advance(b, lats, (8, 3, 17, 6, 1, 9, 2, 8))
    b.close()


@pytest.mark.parametrize("sizes", [[(3000, 3)] * 40, [(3000, 3)] * 300, [(600 + i, 3 + i % 3) for i in range(60)],
                                   [(3, 3000)] * 60])
def test_flat_and_narrow_batches(sizes):
    b, lats = _start(sizes)
    _advance(b, lats, (3, 8, 4, 1, 2))
    b.close()
