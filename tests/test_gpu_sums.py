"""The FP64 sums of a step and of moments() against torch's FP64 sum of the
stored populations with the weights 1, v_x, v_y, |v|^2 (and v_z), on lattices
of more row tiles than the library's scratch holds partials of (8192 in 1D and
2D, 6553 in 3D), where workgroups walk several or, in 1D, the partials go to an
allocation, and of fewer.  FP64 storage (the FP32 forms add up the populations
of one node in FP32).

Tolerance: a chain of n additions in FP64 is off by at most n u sum |w f|, u =
2^-53.  A lane adds fewer than 64 populations per tile of at most two, a tree of
8 follows, and the last pass is compensated; torch's sums take chains of a few
hundred.  512 u on either side: 1024 u in all."""
import threading

import numpy as np
import pytest
import torch

from paper_1402_5487_amd import _plbm, inputs
from paper_1402_5487_amd.lattice import Lattice, Lattice3

pytestmark = pytest.mark.gpu

TOL = 1024 * 2.0 ** -53
V49 = (0, 1, -1, 2, -2, 3, -3)


def _want(P, vel):
    """(sums, sums of magnitudes) of populations (k, nodes), velocities (k, dim)."""
    c = torch.tensor(vel, dtype=torch.float64, device=P.device)
    w = [torch.ones_like(c[:, 0]), c[:, 0], c[:, 1] if c.shape[1] > 1 else 0 * c[:, 0], (c * c).sum(1)]
    if c.shape[1] == 3:
        w.append(c[:, 2])
    per, mag = P.sum(1), P.abs().sum(1)
    return (np.array([float((per * a).sum()) for a in w]), np.array([float((mag * a.abs()).sum()) for a in w]))


def _close(got, P, vel):
    want, mag = _want(P, vel)
    assert np.all(np.abs(np.array(got) - want) <= TOL * mag + 1e-300), (got, want)


@pytest.mark.parametrize("v,kw,th", [((0, 1, -1, 3, -3), {}, 0.35), ((0, 1, -1), dict(zeta=4.0), 0.25),
                                     (V49, dict(velocities=V49, theta0=1.0), 1.0)])
@pytest.mark.parametrize("nx,ny", [(257, 4200), (300, 37)])
def test_sums_of_sheets(v, kw, th, nx, ny):
    lat = Lattice(2, nx, ny, omega=1.7, storage="f64", **kw)
    lat.init(*inputs.random_fields(nx, ny, seed=nx, theta=(th, th), u=0.03))
    vel = [(a, b) for b in v for a in v]
    q = len(vel)
    got = lat.step(3, sums=True)
    P = lat.f.double().view(ny, q, nx).transpose(0, 1).reshape(q, -1)
    _close(got, P, vel)
    _close(lat.sums(), P, vel)          # the pull moves populations, their sums stay


@pytest.mark.parametrize("nx,ny,nz", [(30, 165, 163), (20, 9, 8)])
def test_sums_of_boxes(nx, ny, nz):
    lat = Lattice3(nx, ny, nz, omega=1.4, storage="f64")
    g = torch.Generator().manual_seed(nx)
    lat.init(*(c + a * torch.rand(nz, ny, nx, generator=g, dtype=torch.float64)
               for c, a in ((1.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.4, 0.01))))
    v = (0, 1, -1, 3, -3)
    vel = [(a, b, c) for c in v for b in v for a in v]
    got = lat.step(2, sums=True)
    P = lat.f.double().view(nz * ny, 125, nx).transpose(0, 1).reshape(125, -1)
    _close(got, P, vel)
    _close(lat.sums(), P, vel)


@pytest.mark.parametrize("nx", [1000, 8192 * 256 + 300])
def test_sums_of_tubes(nx):
    lat = Lattice(1, nx, omega=1.1, storage="f64")
    g = torch.Generator().manual_seed(1)
    rho, ux, t = (c + a * torch.rand(nx, generator=g, dtype=torch.float64)
                  for c, a in ((1.0, 0.05), (0.0, 0.02), (0.4, 0.01)))
    lat.init(rho, ux, None, t)
    got = lat.step(5, sums=True)
    P = lat.f.view(5, nx + 6)[:, 3:-3]
    _close(got, P, [(a,) for a in (0, 1, -1, 3, -3)])


def test_sums_while_another_call_holds_the_scratch():
    """A thread asks for sums after every step of a larger lattice; the calls
    beside it find its scratch free or held and are right either way."""
    big = Lattice(2, 1024, 900, omega=1.7).init(*inputs.random_fields(1024, 900, seed=1))
    lat = Lattice(2, 257, 300, omega=1.7).init(*inputs.random_fields(257, 300, seed=2))
    stop, v = threading.Event(), (0, 1, -1, 3, -3)
    torch.cuda.synchronize()

    def hold():
        with torch.cuda.stream(torch.cuda.Stream()):
            while not stop.is_set():
                big.step(10, sums=True)

    t = threading.Thread(target=hold)
    t.start()
    try:
        for _ in range(40):
            got = lat.step(2, sums=True)
            _close(got, lat.f.view(300, 25, 257).transpose(0, 1).reshape(25, -1), [(a, b) for b in v for a in v])
    finally:
        stop.set()
        t.join()


@pytest.mark.parametrize("nx,ny,nz", [(30, 165, 163), (20, 9, 8), (256, 6, 5)])
def test_sums_of_fp32_boxes(nx, ny, nz):
    """A node's sums are taken in FP32: fewer than 130 additions and products, each
    off by at most 2^-24."""
    lat = Lattice3(nx, ny, nz, omega=1.4, storage="f32")
    g = torch.Generator().manual_seed(nx)
    lat.init(*(c + a * torch.rand(nz, ny, nx, generator=g, dtype=torch.float64)
               for c, a in ((1.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.4, 0.01))))
    v = (0, 1, -1, 3, -3)
    got = np.array(lat.step(2, sums=True))
    P = lat.f.double().view(nz * ny, 125, nx).transpose(0, 1).reshape(125, -1)
    want, mag = _want(P, [(a, b, c) for c in v for b in v for a in v])
    assert np.all(np.abs(got - want) <= 130 * 2.0 ** -24 * mag), (got, want)


def test_noalloc_sums_of_more_tiles_than_the_scratch_holds():
    lat = Lattice(2, 257, 4200, omega=1.7).init(*inputs.random_fields(257, 4200, seed=3))
    a, b = lat.f.clone(), torch.empty_like(lat.f)
    got = _plbm.step_noalloc(lat.desc, a, b, 1, True, lat.stream)
    v = (0, 1, -1, 3, -3)
    _close(got, b.view(4200, 25, 257).transpose(0, 1).reshape(25, -1), [(x, y) for y in v for x in v])
