"""How the fused steps cut a lattice (CPU): every node of it is written by
exactly one lane of one launch, whatever the size and the model."""
import ctypes
import re

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


# what a step of its own launches
SINGLE = {"k_step2d", "k_step2d_fields", "k_step_q9", "k_step_gen2d", "k_step1d", "k_step_q3_1d", "k_step_gen1d",
          "k_step3d"}
SIZES = {1: [(7, 1), (1000, 1), (1025, 1), (70000, 1)],
         2: [(8, 9), (64, 64), (129, 127), (300, 400), (28, 10000), (900, 1300), (1501, 1100)]}


@pytest.mark.parametrize("model,storage,entry", [
    (m, st, e) for m, st in FORMS + [("d1q5", "f64"), ("d1q3", "f32"), ("d1q7", "f64")]
    for e in ("plbm_step", "plbm_advance", "plbm_step_noalloc") if e != "plbm_step_noalloc" or m in ("d2q25", "d1q5")])
def test_launches_hand_the_state_on_and_end_where_steps_do(recorder, model, storage, entry):  # noqa: F811
    """Each launch reads what the one before wrote (a 1D lattice in place too),
    the last writes the buffer that the number of steps says, and of the calls
    that keep the state before it is a single step."""
    dim = int(model[1])
    tube = {"d1q5": lambda nx, ny, st: _plbm.desc_default(1, nx, 1, 1.2, st),
            "d1q3": lambda nx, ny, st: _plbm.desc_q3(1, nx, 1, 1.2, st, zeta=4.0),
            "d1q7": lambda nx, ny, st: _plbm.desc_general(1, nx, 1, 1.2, st, V49, 1.0)}
    for nx, ny in SIZES[dim]:
        d = (MODELS.get(model) or tube[model])(nx, ny, storage)
        for n in list(range(1, 14)) + [40, 41]:
            for sums in (False, True):
                at = 0x1000
                ls = [x for x in recorder.step(d, n, entry, sums) if x.kernel != "k_reduce_partials"]
                for x in ls:
                    assert x.src == at and x.block <= 1024 and x.lds <= 160 * 1024, (nx, ny, n, x.name)
                    at = x.dst
                assert at == (0x1000 if n % 2 == 0 else 0x2000), (nx, ny, n)
                if entry != "plbm_advance":
                    last = ls[-1]
                    assert last.src != last.dst
                    assert last.kernel in SINGLE, (nx, ny, n, last.name)


@pytest.mark.parametrize("nx,ny", [(4096, 4096), (257, 4200), (64, 64)])
@pytest.mark.parametrize("model,storage", [f for f in FORMS if f[1] != "f16dev"])
def test_sums_keep_to_the_scratch(recorder, model, storage, nx, ny):  # noqa: F811
    """At most as many workgroups as the scratch holds partials of, which walk the
    row tiles, and nothing allocated."""
    recorder.lib.rec_allow_mallocs(0)
    last = [x for x in recorder.step(MODELS[model](nx, ny, storage), 2, sums=True) if x.kernel in SINGLE][-1]
    recorder.lib.rec_allow_mallocs(-1)
    assert last.grid == min(8192, -(-nx // 256) * ny)


TUBES = {"d1q5": lambda nx, st: _plbm.desc_default(1, nx, 1, 1.2, st),
         "d1q3": lambda nx, st: _plbm.desc_q3(1, nx, 1, 1.2, st, zeta=4.0),
         "d1q7": lambda nx, st: _plbm.desc_general(1, nx, 1, 1.2, st, V49, 1.0)}


@pytest.mark.parametrize("model,storage", [("d1q5", "f64"), ("d1q3", "f32"), ("d1q7", "f64")])
@pytest.mark.parametrize("nx", [1, 64, 1000, 1024, 1025, 20000])
@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 4098, 8192, 8193, 100001, 2 ** 31 - 1])
def test_long_calls_of_a_tube_are_short_launches(recorder, model, storage, nx, n):  # noqa: F811
    """No launch takes more than 4096 steps, together they take all of them, and
    the halo of a tile (three nodes a step) stays a small number."""
    if n > 10 ** 6 and (nx, model) != (64, "d1q5"):
        n = 10 ** 5 + 7                                # up to tens of millions of launches otherwise
    at, taken = 0x1000, 0
    for x in recorder.step(TUBES[model](nx, storage), n, "plbm_advance"):
        steps = x.extra[2] if x.kernel == "k_tube" else 1
        assert x.kernel in ("k_tube", *SINGLE) and x.src == at and 1 <= steps <= 4096
        assert x.src != x.dst or steps % 2 == 0
        at, taken = x.dst, taken + steps
    assert taken == n and at == (0x1000 if n % 2 == 0 else 0x2000)


# (model, storage, nx, ny, steps): measured at up to five times the single steps
# on tiles or strips
FLAT = [("d2q25", "f16dev", 100000, 3, 20), ("d2q25", "f16dev", 10000, 24, 3), ("d2q25", "f16dev", 113, 3000, 3), ("d2q25", "f64", 10000, 3, 20),
        ("d2q25", "f32", 30000, 3, 4), ("d2q16", "f32", 30000, 3, 20),
        ("d2q49", "f32", 10000, 3, 20), ("d2q49", "f64", 300000, 3, 20), ("d2q49", "f64", 100000, 3, 4)]
# no tiles there: strips are faster than single steps
FLAT_STRIPS = [("d2q25", "f64", 100000, 4, 4), ("d2q25", "f32", 300000, 3, 20), ("d2q9", "f64", 300000, 3, 20),
               ("d2q9", "f32", 300000, 3, 20), ("d2q16", "f32", 100000, 3, 20), ("d2q16", "f64", 300000, 3, 20)]
# and these stay
TILED = [("d2q25", "f64", 256, 256, 6), ("d2q25", "f16dev", 700, 900, 4), ("d2q25", "f32", 1000, 1000, 4),
         ("d2q25", "f64", 3, 30000, 4), ("d2q25", "f32", 3000, 3, 6), ("d2q9", "f32", 1000, 1000, 10),
         ("d2q16", "f64", 1000, 900, 4), ("d2q49", "f32", 500, 500, 4), ("d2q49", "f64", 500, 500, 4)]


@pytest.mark.parametrize("model,storage,nx,ny,n", FLAT)
def test_flat_lattices_take_single_steps(recorder, model, storage, nx, ny, n):  # noqa: F811
    assert {x.kernel for x in recorder.step(MODELS[model](nx, ny, storage), n, "plbm_advance")} <= SINGLE


@pytest.mark.parametrize("model,storage,nx,ny,n", FLAT_STRIPS)
def test_long_flat_lattices_take_strips(recorder, model, storage, nx, ny, n):  # noqa: F811
    assert {x.kernel for x in recorder.step(MODELS[model](nx, ny, storage), n, "plbm_advance")} & STRIPS
    assert "k_tile" not in {x.kernel for x in recorder.step(MODELS[model](nx, ny, storage), n, "plbm_advance")}


@pytest.mark.parametrize("model,storage,nx,ny,n", TILED)
def test_other_lattices_keep_their_tiles(recorder, model, storage, nx, ny, n):  # noqa: F811
    assert {x.kernel for x in recorder.step(MODELS[model](nx, ny, storage), n, "plbm_advance")} == {"k_tile"}


@pytest.mark.parametrize("nx,ny,w", [(240, 4700, 240), (241, 4700, 241), (480, 2353, 240), (960, 1200, 240),
                                     (961, 1300, 208), (1200, 900, 240), (1201, 1000, 208)])
def test_whole_strips_take_three_steps(recorder, nx, ny, w):  # noqa: F811
    got = recorder.step(MODELS["d2q25"](nx, ny, "f32"), 9, "plbm_advance")
    assert len(got) == 3 and {(x.kernel, x.extra[2]) for x in got} == {("k_step2d_sweep", w)}


@pytest.mark.parametrize("nx,ny", [(27000, 64), (30000, 48), (55000, 40)])
def test_strips_fill_their_rounds(recorder, nx, ny):  # noqa: F811
    """D2Q49 FP64 has more strips than the 256 workgroups that run at once: the
    rounds take fewer rows one after another than whole strips would (halo: three
    rows at either end)."""
    x = recorder.step(MODELS["d2q49"](nx, ny, "f64"), 4, "plbm_advance")[0]
    strips, chunks, _, h, _, per, wgs = x.extra
    assert x.kernel == "k_pair_gen" and strips > 256 and per == 1
    assert -(-wgs // 256) * (h + 6) < -(-strips // 256) * (ny + 6)
    assert (_owners(recorder, x, nx, ny) == 1).all()


# (model, storage, nx, ny, whether single steps store non-temporally): rows on
# half lines; ragged ones of which two buffers just fill L2; ragged ones
@pytest.mark.parametrize("model,storage,nx,ny,nt", [
    ("d2q25", "f16dev", 3008, 700, True), ("d2q25", "f16dev", 30000, 6, True), ("d2q25", "f64", 3001, 16, True),
    ("d2q16", "f32", 30001, 6, True), ("d2q49", "f32", 1501, 33, True), ("d2q9", "f64", 30001, 6, True),
    ("d2q25", "f16dev", 30000, 13, False), ("d2q25", "f32", 1501, 66, False), ("d2q9", "f64", 1501, 66, False),
    ("d2q16", "f32", 3000, 66, False), ("d2q49", "f64", 1501, 33, False)])
def test_stores_of_single_steps(recorder, model, storage, nx, ny, nt):  # noqa: F811
    x, = recorder.step(MODELS[model](nx, ny, storage), 1)
    last = re.search(r"Lb([01])EEEv", x.name)          # the last template argument
    assert x.kernel in SINGLE and last.group(1) == str(int(nt)), x.name


@pytest.mark.parametrize("model,storage", [("d1q5", "f64"), ("d1q3", "f32"), ("d1q7", "f64")])
@pytest.mark.parametrize("nx,n,entry,kernels", [
    (1000, 1, "plbm_advance", 1), (1000, 2, "plbm_step", 2), (3000, 2, "plbm_advance", 2), (40_000_000, 1, "plbm_step", 1),
    (150_000, 1, "plbm_advance", 1)])
def test_launches_of_one_step_of_a_tube_are_single_steps(recorder, model, storage, nx, n, entry, kernels):  # noqa: F811
    ls = recorder.step(TUBES[model](nx, storage), n, entry)
    assert [x.kernel in SINGLE for x in ls] == [True] * kernels


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nx", [16, 256, 250])
def test_a_box_with_sums_leaves_lds_for_them(recorder, nx, storage):  # noqa: F811
    """The block sums hold five doubles a wave of a workgroup's four beside what
    the launch reserves; a CU has 160 KB."""
    d = _plbm.desc_3d(nx, 8, 8, 1.2, storage)
    one, last = [x for x in recorder.step(d, 2, sums=True) if x.kernel == "k_step3d"]
    assert one.lds <= 160 * 1024 and last.lds + 5 * 4 * 8 <= 160 * 1024


@pytest.mark.parametrize("nx,ny,nz,grid", [
    (16, 16, 16, 256), (3, 3, 3, 9), (128, 16, 16, 256), (300, 16, 8, 256),     # whole rows, at most one per CU
    (16, 16, 17, 68), (30, 30, 30, 225), (129, 16, 17, 204),                    # four segments a workgroup
    (256, 20, 20, 400)])                                                        # whole rows that fill it
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_workgroups_of_a_box(recorder, nx, ny, nz, grid, storage):  # noqa: F811
    d = _plbm.desc_3d(nx, ny, nz, 1.2, storage)
    assert [x.grid for x in recorder.step(d, 2)] == [grid] * 2


@pytest.mark.parametrize("nx,ny,nz,grid", [(16, 16, 16, 256), (20, 20, 20, 100), (256, 20, 20, 400)])
def test_workgroups_of_fields_of_a_box(recorder, nx, ny, nz, grid):  # noqa: F811
    """Initial states and moments are cut as the step is."""
    d = _plbm.desc_3d(nx, ny, nz, 1.2, "f64")
    at = [ctypes.c_void_p(0x1000 * (i + 1)) for i in range(6)]
    recorder.lib.rec_clear()
    assert recorder.lib.plbm_init3(ctypes.byref(d), *at, None) == _plbm.PLBM_OK
    assert recorder.lib.plbm_moments3(ctypes.byref(d), *at, None, None) == _plbm.PLBM_OK
    assert [(x.kernel, x.grid) for x in recorder.launches()] == [("k_init3d", grid), ("k_moments3d", grid)]
