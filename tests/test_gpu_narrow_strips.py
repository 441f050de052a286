"""Fused steps on rows that close on themselves, one to four chunks side by
side in a workgroup, against the same steps one by one.  Both round the same
operations in the same order: equal bit for bit, the tolerance is zero."""
import pytest
import torch

from paper_1402_5487_amd import inputs
from paper_1402_5487_amd.lattice import Lattice, Lattice3

pytestmark = pytest.mark.gpu


# D2Q49: a lane holds one of 112 (FP64) or 232 (FP32) columns of two or four
# waves; D2Q16 one of 256.  At, below and past what lets chunks share them.
@pytest.mark.parametrize("v,theta,least,widths", [
    ((0, 1, -1, 2, -2, 3, -3), 1.0, 1 << 18, (16, 24, 28, 29, 32, 33, 56, 57, 58, 59, 112, 116)),
    ((1, -1, 3, -3), 4.0 / 3.0, 1 << 20, (32, 64, 65, 128))])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_chunks_side_by_side_equal_single_steps(v, theta, least, widths, storage):
    for nx in widths:
        ny = least // nx + 5
        fields = inputs.random_fields(nx, ny, seed=nx, theta=(theta, theta), u=0.03)
        a, b = (Lattice(2, nx, ny, omega=1.6, storage=storage, velocities=v, theta0=theta).init(*fields)
                for _ in range(2))
        for n in (5, 4, 2):
            a.step(n)
        for _ in range(11):
            b.step(1)
        assert torch.equal(a.f, b.f) and a.cur == b.cur, (nx, ny)


@pytest.mark.parametrize("nx,storage", [(64, "f64"), (200, "f32"), (1000, "f64")])
def test_a_long_call_of_a_tube_equals_short_ones(nx, storage):
    """More steps than one launch takes (4096), in place and into the other
    buffer: 8193 and then 8192 of them against calls of 127."""
    rho, ux, _, th = inputs.shock_tube(nx, rho_r=0.7)
    a, b = (Lattice(1, nx, omega=1.1, storage=storage).init(rho, ux, None, th) for _ in range(2))
    for n in (8193, 8192):
        a.step(n)
    for _ in range((8193 + 8192) // 127):
        b.step(127)
    b.step((8193 + 8192) % 127)
    assert torch.equal(a.f, b.f) and a.cur == b.cur


# flat lattices: tiles, strips and single steps as they pay
@pytest.mark.parametrize("nx,ny", [(3000, 20), (10000, 3), (10000, 24), (30000, 4), (100000, 3), (300000, 3), (30000, 48)])
@pytest.mark.parametrize("kw,theta,storage", [({}, 0.4, "f64"), ({}, 0.4, "f32"), ({}, 0.35, "f16dev"),
                                              (dict(zeta=4.0), 0.25, "f32"), (dict(zeta=4.0), 0.25, "f64"),
                                              (dict(velocities=(1, -1, 3, -3), theta0=4.0 / 3.0), 4.0 / 3.0, "f32"),
                                              (dict(velocities=(0, 1, -1, 2, -2, 3, -3), theta0=1.0), 1.0, "f64")])
def test_flat_lattices_equal_single_steps(nx, ny, kw, theta, storage):
    fields = inputs.random_fields(nx, ny, seed=nx + ny, theta=(theta, theta), u=0.03)
    a, b = (Lattice(2, nx, ny, omega=1.6, storage=storage, **kw).init(*fields) for _ in range(2))
    for n in (3, 4, 12):
        a.step(n)
    for _ in range(19):
        b.step(1)
    assert torch.equal(a.f, b.f) and a.cur == b.cur


# boxes of at most 256 rows take whole rows, larger ones four segments a
# workgroup: a box and four copies of it, along z, keep the same state
@pytest.mark.parametrize("nx,ny,nz", [(16, 16, 16), (3, 5, 7), (129, 8, 20), (300, 9, 14), (70, 11, 13)])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_small_boxes_equal_their_doubles(nx, ny, nz, storage):
    g = torch.Generator().manual_seed(nx)
    fields = [c + a * torch.rand(nz, ny, nx, generator=g, dtype=torch.float64)
              for c, a in ((1.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.4, 0.01))]
    a, b = (Lattice3(nx, ny, n, omega=1.2, storage=storage) for n in (nz, 4 * nz))
    a.init(*fields)
    b.init(*(f.repeat(4, 1, 1) for f in fields))
    sa, sb = a.step(3, sums=True), b.step(3, sums=True)
    assert torch.equal(b.f.view(4, -1), a.f.view(1, -1).expand(4, -1))
    assert all(abs(4 * x - y) <= 1e-12 * 4 * abs(sa[0]) for x, y in zip(sa, sb))
