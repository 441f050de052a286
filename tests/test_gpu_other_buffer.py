"""plbm_step, plbm_step_fields and plbm_step_noalloc leave the state one step
before in the buffer that does not hold the result; plbm_advance and
plbm_advance_fields give the same result.  Against single steps, bit for bit
(the tolerance is zero)."""
import ctypes

import pytest
import torch

from paper_1402_5487_amd import _plbm, inputs
from paper_1402_5487_amd.lattice import Lattice, Lattice3

pytestmark = pytest.mark.gpu

V49 = (0, 1, -1, 2, -2, 3, -3)
KINDS = {
    "d2q25": (dict(), 0.35), "d2q9": (dict(zeta=4.0), 0.25),
    "d2q16": (dict(velocities=(1, -1, 3, -3), theta0=4.0 / 3.0), 4.0 / 3.0),
    "d2q49": (dict(velocities=V49, theta0=1.0), 1.0),
}
# tiles of each depth, strips, single steps
CASES = [("d2q25", 64, 64, "f64"), ("d2q25", 300, 37, "f16dev"), ("d2q25", 401, 257, "f32"),
         ("d2q25", 257, 4100, "f64"), ("d2q25", 257, 4100, "f32"), ("d2q25", 1501, 1100, "bf16dev"),
         ("d2q9", 128, 128, "f64"), ("d2q9", 1501, 700, "f32"), ("d2q16", 300, 270, "f32"),
         ("d2q16", 1025, 1030, "f64"), ("d2q49", 64, 60, "f64"), ("d2q49", 700, 400, "f32"), ("d2q49", 28, 10000, "f64")]


def _states(lat, n):
    """The buffers' contents after 0 .. n single steps."""
    out = [lat.f.clone()]
    for _ in range(n):
        lat.step(1)
        out.append(lat.f.clone())
    return out


def _check(call, want, n, same=True):
    a, b = want[0].clone(), torch.full_like(want[0], float("nan"))
    call(a, b, n)
    new, old = (a, b) if n % 2 == 0 else (b, a)
    assert torch.equal(new, want[n]), n
    if same:
        assert torch.equal(old, want[n - 1]), n


@pytest.mark.parametrize("model,nx,ny,storage", CASES)
def test_the_other_buffer_holds_the_state_before(model, nx, ny, storage):
    kw, th = KINDS[model]
    lat = Lattice(2, nx, ny, omega=1.6, storage=storage, **kw)
    want = _states(lat.init(*inputs.random_fields(nx, ny, seed=nx, theta=(th, th), u=0.03)), 12)
    d, st = lat.desc, lat.stream
    for n in (1, 2, 3, 4, 5, 7, 9, 12):
        for sums in (False, True):
            _check(lambda a, b, n: _plbm.step(d, a, b, n, sums, st), want, n)
            _check(lambda a, b, n: _plbm.advance(d, a, b, n, sums, st), want, n, same=False)
            if model == "d2q25":
                _check(lambda a, b, n: _plbm.step_noalloc(d, a, b, n, sums, st), want, n)
        if model == "d2q25":
            out = [torch.empty(ny, nx, dtype=torch.float64, device="cuda") for _ in range(4)]
            _check(lambda a, b, n: _plbm.step_fields(d, a, b, n, *out, st), want, n)
            _check(lambda a, b, n: _plbm.advance_fields(d, a, b, n, *out, st), want, n, same=False)


@pytest.mark.parametrize("nx", [3, 1000, 1025, 5001])
@pytest.mark.parametrize("kw,storage", [({}, "f64"), ({}, "f32"), (dict(zeta=4.0), "f64"),
                                        (dict(velocities=V49, theta0=1.0), "f32")])
def test_the_other_buffer_of_a_tube(nx, kw, storage):
    g = torch.Generator().manual_seed(nx)
    th = {0: 0.4, 1: 0.25, 2: 1.0}[len(kw)]
    rho, ux, t = (c + a * torch.rand(nx, generator=g, dtype=torch.float64)
                  for c, a in ((1.0, 0.05), (0.0, 0.02), (th, 0.01)))
    lat = Lattice(1, nx, omega=1.1, storage=storage, **kw)
    want = _states(lat.init(rho, ux, None, t), 41)
    for n in (1, 2, 3, 8, 40, 41):
        for sums in (False, True):
            _check(lambda a, b, n: _plbm.step(lat.desc, a, b, n, sums, lat.stream), want, n)
            _check(lambda a, b, n: _plbm.advance(lat.desc, a, b, n, sums, lat.stream), want, n, same=False)


def test_the_other_buffer_of_a_box():
    lat = Lattice3(20, 7, 5, omega=1.2, storage="f64")
    g = torch.Generator().manual_seed(1)
    lat.init(*(c + a * torch.rand(5, 7, 20, generator=g, dtype=torch.float64)
               for c, a in ((1.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.4, 0.01))))
    want = _states(lat, 4)
    for n in (1, 2, 3, 4):
        for sums in (False, True):
            _check(lambda a, b, n: _plbm.step(lat.desc, a, b, n, sums, lat.stream), want, n)
            _check(lambda a, b, n: _plbm.advance(lat.desc, a, b, n, sums, lat.stream), want, n)


def test_advance_refuses_what_step_refuses():
    lib = _plbm.lib
    d = _plbm.desc_default(2, 64, 64, 1.5, "f64")
    a, b = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x2000)
    assert lib.plbm_advance(ctypes.byref(d), a, a, 1, None, None) == _plbm.PLBM_EINVAL
    assert lib.plbm_advance(ctypes.byref(d), a, b, -1, None, None) == _plbm.PLBM_EINVAL
    assert lib.plbm_advance_fields(ctypes.byref(d), a, b, 0, None, None, None, None, None) == _plbm.PLBM_EINVAL
