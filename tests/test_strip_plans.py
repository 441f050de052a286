"""How the fused steps cut a lattice (CPU): every node of it is written by
exactly one lane of one launch, whatever the size and the model."""
import ctypes

import numpy as np
import pytest

from launches import recorder  # noqa: F401  (fixture)
from paper_1402_5487_amd import _plbm

V49 = (0, 1, -1, 2, -2, 3, -3)
MODELS = {
    "d2q25": lambda nx, ny, st: _plbm.desc_default(2, nx, ny, 1.6, st),
    "d2q9": lambda nx, ny, st: _plbm.desc_q3(2, nx, ny, 1.6, st, zeta=4.0),
    "d2q16": lambda nx, ny, st: _plbm.desc_general(2, nx, ny, 1.6, st, (1, -1, 3, -3), 4.0 / 3.0),
    "d2q49": lambda nx, ny, st: _plbm.desc_general(2, nx, ny, 1.6, st, V49, 1.0),
}
FORMS = [("d2q25", "f64"), ("d2q25", "f32"), ("d2q25", "f16dev"), ("d2q9", "f64"), ("d2q9", "f32"),
         ("d2q16", "f64"), ("d2q16", "f32"), ("d2q49", "f64"), ("d2q49", "f32")]
STRIPS = {"k_step2d_sweep", "k_sweep_q9", "k_pair_gen"}


def _owners(rec, launch, nx, ny):
    """How many lanes write each node, wave by wave as the kernel places them."""
    strips, chunks, w, h, span, per, wgs = launch.extra
    assert launch.grid == wgs and launch.block % 64 == 0
    grid = (ctypes.c_int * 7)(*launch.extra)
    share = launch.block // per                        # lanes of one chunk
    own = np.zeros((ny, nx), dtype=np.int8)
    for first in range(0, launch.block, 64):
        side = rec.lib.rec_sweep_side(grid, first, launch.block)
        lo, hi = max(0, first - side * share), min(w, first - side * share + 64)
        for b in range(wgs):
            c, xs = b // strips, b % strips * w
            ya = (c * per + side) * h
            own[ya:min(ya + h, ny), xs + lo:max(xs + lo, min(xs + hi, nx))] += 1
    return own


@pytest.mark.parametrize("model,storage", FORMS)
@pytest.mark.parametrize("nx", [16, 24, 28, 29, 32, 33, 56, 57, 58, 59, 63, 64, 65, 112, 113, 116, 117, 128, 129,
                                232, 233, 256, 257, 449])
def test_strips_write_every_node_once(recorder, model, storage, nx):  # noqa: F811
    for ny in (1 + (1 << 21) // nx, 20011):
        seen = 0
        for launch in recorder.step(MODELS[model](nx, ny, storage), 12):
            if launch.kernel in STRIPS and seen < 2:
                own = _owners(recorder, launch, nx, ny)
                assert own.min() == 1 and own.max() == 1, (ny, launch.extra, launch.block)
                seen += 1
