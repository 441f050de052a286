"""Several steps fused into one launch against the same steps launched one by
one.  Both round the same operations in the same order and hold the values
between the steps in the storage type, so every population must be equal bit
for bit; the tolerance is zero."""
import pytest
import torch

from paper_1402_5487_amd import inputs
from paper_1402_5487_amd.batch import Batch
from paper_1402_5487_amd.lattice import Lattice, Lattice3

pytestmark = pytest.mark.gpu


def _pair(make, fields, split, whole):
    """Two lattices of one state: one stepped step by step, one in calls of `whole`."""
    a, b = make().init(*fields), make().init(*fields)
    for n in whole:
        a.step(n)
    for _ in range(split):
        b.step(1)
    return a, b


# tiles: the largest lattices of 8 x 8, 16 x 16 and 20 x 20 nodes a tile, one more
# row or column than that, ragged edges, fewer nodes than a tile and than its
# margin, long thin ones; every remainder of the steps
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 700), (64, 64), (128, 128), (129, 127), (256, 256), (300, 37),
                                   (257, 250), (320, 320), (401, 257), (701, 3)])
@pytest.mark.parametrize("storage,rounding", [("f64", "nearest"), ("f32", "nearest"), ("f16dev", "nearest"),
                                              ("bf16dev", "nearest"), ("f16dev", "stochastic"),
                                              ("bf16dev", "stochastic")])
def test_fused_small_steps_equal_single_steps(nx, ny, storage, rounding):
    fields = inputs.random_fields(nx, ny, seed=nx + ny)
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.7, storage=storage, rounding=rounding, theta0=0.35),
                 fields, 28, (2, 3, 5, 8, 10))
    assert torch.equal(a.f, b.f) and a.cur == b.cur
    got, want = a.step_fields(6), b.step_fields(1)
    for _ in range(5):
        b.step(1)
    assert torch.equal(a.f, b.f) and all(torch.equal(g, w) for g, w in zip(got, want))
    s = a.step(8, sums=True)
    for _ in range(7):
        b.step(1)
    assert s == b.step(1, sums=True) and torch.equal(a.f, b.f)


# one strip of up to 256 columns that closes on itself, with four, two or one
# chunk side by side; strips of 224 (FP32) and 240 (FP64) columns beyond: at
# and past their multiples, ragged rows, a last strip of a single column, more
# rows than a chunk and fewer than its halo
@pytest.mark.parametrize("nx,ny", [(63, 16700), (64, 16401), (65, 16200), (128, 8201), (256, 4101), (257, 4100),
                                   (448, 2353), (449, 2340), (1501, 707), (16385, 65), (104850, 11)])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_fused_steps_equal_single_steps(nx, ny, storage):
    fields = inputs.random_fields(nx, ny, seed=nx + ny)
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.7, storage=storage), fields, 11, (5, 4, 2))
    assert torch.equal(a.f, b.f) and a.cur == b.cur


# FP32 in threes (strips of up to 240 columns) and, where those do not fill the
# lanes, in pairs: closed strips with one, two and four chunks side by side, ragged
# rows, one chunk that is the whole height; every remainder of the steps, with
# fields and with sums
@pytest.mark.parametrize("nx,ny", [(64, 17000), (63, 17001), (128, 8300), (224, 4700), (256, 4101), (448, 2353),
                                   (673, 1600), (1501, 707), (1121, 940), (16385, 65), (57344, 19)])
def test_three_fused_steps_equal_single_steps(nx, ny):
    fields = inputs.random_fields(nx, ny, seed=nx + ny)
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.7, storage="f32"), fields, 30, (3, 6, 7, 14))
    assert torch.equal(a.f, b.f) and a.cur == b.cur
    got, want = a.step_fields(9), b.step_fields(1)
    for _ in range(8):
        b.step(1)
    assert torch.equal(a.f, b.f) and all(torch.equal(g, w) for g, w in zip(got, want))
    s = a.step(10, sums=True)
    for _ in range(9):
        b.step(1)
    assert s == b.step(1, sums=True) and torch.equal(a.f, b.f)


# widths that FP32 threes take in whole strips of 240 columns, and one column more
# (a closed strip of 241, five and six of 208)
@pytest.mark.parametrize("nx,ny", [(240, 4700), (241, 4700), (480, 2353), (960, 1200), (961, 1300), (1200, 900),
                                   (1201, 1000)])
def test_three_fused_steps_of_whole_strips_equal_single_steps(nx, ny):
    fields = inputs.random_fields(nx, ny, seed=nx + ny)
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.7, storage="f32"), fields, 14, (9, 3, 2))
    assert torch.equal(a.f, b.f) and a.cur == b.cur


@pytest.mark.parametrize("nx,ny", [(1501, 1100), (1345, 1121), (224, 6700), (128, 11730)])
@pytest.mark.parametrize("storage,rounding", [("f16dev", "nearest"), ("bf16dev", "nearest"),
                                              ("f16dev", "stochastic"), ("bf16dev", "stochastic")])
def test_fused_16_bit_steps_equal_single_steps(nx, ny, storage, rounding):
    fields = inputs.random_fields(nx, ny, seed=nx)
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.7, storage=storage, rounding=rounding, theta0=0.35),
                 fields, 8, (8,))
    assert torch.equal(a.f, b.f)


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_fused_steps_with_fields_and_sums(storage):
    """The first of the fused steps writes the fields of the state it reads;
    a step that takes sums comes after fused ones."""
    nx, ny = 1050, 1002
    fields = inputs.random_fields(nx, ny, seed=5)
    a, b = (Lattice(2, nx, ny, omega=1.7, storage=storage).init(*fields) for _ in range(2))
    got, want = a.step_fields(7), b.step_fields(1)
    for _ in range(6):
        b.step(1)
    assert torch.equal(a.f, b.f)
    assert all(torch.equal(g, w) for g, w in zip(got, want))
    s, t = a.step(6, sums=True), None
    for _ in range(6):
        t = b.step(1, sums=True)
    assert torch.equal(a.f, b.f) and s == t


def test_fused_steps_in_a_graph():
    """Captured once, replayed between eager work: every replay as eager."""
    nx, ny = 700, 1502
    fields = inputs.random_fields(nx, ny, seed=2)
    a, b = (Lattice(2, nx, ny, omega=1.7, storage="f32").init(*fields) for _ in range(2))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            a.step(4)
    torch.cuda.current_stream().wait_stream(s)
    for _ in range(3):
        g.replay()
        b.step(4)
        torch.cuda.synchronize()
        assert torch.equal(a.f, b.f)


# D2Q9: tiles of nine, seven and five steps, then three, then one; beyond them
# strips of four (FP64) or five (FP32); every remainder, fewer rows than the halo
@pytest.mark.parametrize("nx,ny", [(3, 3), (16, 5), (17, 4), (31, 9), (128, 128), (129, 128), (256, 255), (257, 256),
                                   (700, 50), (1025, 3), (16, 65600), (17, 62000), (224, 4701), (225, 4700),
                                   (241, 4400), (1501, 700), (262144, 5)])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_fused_d2q9_steps_equal_single_steps(nx, ny, storage):
    fields = inputs.random_fields(nx, ny, seed=nx + ny, theta=(0.25, 0.25))
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.7, storage=storage, zeta=4.0), fields, 44,
                 (11, 12, 8, 6, 7))
    assert torch.equal(a.f, b.f) and a.cur == b.cur
    s = a.step(9, sums=True)
    for _ in range(8):
        b.step(1)
    assert s == b.step(1, sums=True) and torch.equal(a.f, b.f)


@pytest.mark.parametrize("nx,ny", [(3, 4), (64, 60), (128, 128), (129, 130), (256, 256), (300, 270), (1025, 1030)])
@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("v,theta", [((1, -1, 3, -3), 4.0 / 3.0), ((0, 1, -1, 2, -2, 3, -3), 1.0)])
def test_fused_general_steps_equal_single_steps(nx, ny, storage, v, theta):
    fields = inputs.random_fields(nx, ny, seed=nx + ny, theta=(theta, theta), u=0.03)
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.6, storage=storage, velocities=v, theta0=theta), fields, 11,
                 (5, 4, 2))
    assert torch.equal(a.f, b.f) and a.cur == b.cur


# strips on half lines, of 240 (FP32, threes and pairs) and 104 columns (D2Q49 in
# FP64): at and past their multiples and whole ragged rows
@pytest.mark.parametrize("nx,ny", [(104, 2600), (208, 1300), (209, 1301), (480, 2200), (481, 2190), (720, 1460)])
@pytest.mark.parametrize("storage,v,theta", [("f32", (0, 1, -1, 3, -3), 0.4), ("f64", (0, 1, -1, 2, -2, 3, -3), 1.0)])
def test_fused_steps_on_half_lines_equal_single_steps(nx, ny, storage, v, theta):
    fields = inputs.random_fields(nx, ny, seed=nx + ny, theta=(theta, theta), u=0.03)
    a, b = _pair(lambda: Lattice(2, nx, ny, omega=1.6, storage=storage, velocities=v, theta0=theta), fields, 13,
                 (9, 4))
    assert torch.equal(a.f, b.f) and a.cur == b.cur


# 1D: short lattices in one workgroup (in place for an even number of steps); tiles
# with halos for longer ones, and for many steps of 1000 nodes; the tile that
# leaves one node, fewer nodes than the halo in the last tile; one step, few, many;
# the ghosts belong to the buffer
@pytest.mark.parametrize("nx", [1, 2, 5, 63, 65, 1000, 1024, 1025, 1143, 5001, 70000])
@pytest.mark.parametrize("model,storage", [("d1q5", "f64"), ("d1q5", "f32"), ("d1q3", "f64"), ("d1q3", "f32"),
                                           ("d1q4", "f64"), ("d1q7", "f32"), ("d1q7", "f64")])
def test_fused_tube_steps_equal_single_steps(nx, model, storage):
    kw = {"d1q5": {}, "d1q3": dict(zeta=4.0), "d1q4": dict(velocities=(1, -1, 3, -3), theta0=4.0 / 3.0),
          "d1q7": dict(velocities=(0, 1, -1, 2, -2, 3, -3), theta0=1.0)}[model]
    g = torch.Generator().manual_seed(nx)
    th = {"d1q5": 0.4, "d1q7": 1.0}.get(model, 0.25)
    rho, ux, t = (c + a * torch.rand(nx, generator=g, dtype=torch.float64) for c, a in ((1.0, 0.05), (0.0, 0.02), (th, 0.01)))
    a, b = _pair(lambda: Lattice(1, nx, omega=1.1, storage=storage, **kw), (rho, ux, None, t), 121,
                 (1, 2, 3, 10, 105))
    assert torch.equal(a.f, b.f) and a.cur == b.cur
    s = a.step(5, sums=True)
    for _ in range(4):
        b.step(1)
    assert s == b.step(1, sums=True) and torch.equal(a.f, b.f)


# batches by their size: three steps on tiles of 8 x 8 and 16 x 16, two on
# 16 x 16, strips of three past 2^20 nodes (rows of one, two and four chunks side
# by side, several strips, ragged rows); up to 48 sizes decode arithmetically,
# more go through a list; graph replays, a last fused launch and single steps
MIXED = [(64, 64)] * 20 + [(100, 90)] * 12 + [(256, 250)] * 2 + [(300, 200), (513, 60), (31, 300)]


@pytest.mark.parametrize("sizes", [[(64, 64)] * 3 + [(31, 20)], [(3, 3 + i) for i in range(50)],
                                   [(96, 96)] * 5 + [(33, 65)], [(20 + i % 7, 21 + i) for i in range(50)],
                                   MIXED, [(64 + i, 90 + i) for i in range(50)],
                                   MIXED * 3, [(130 + i, 140 + i) for i in range(50)]])
def test_fused_batch_steps_equal_single_lattices(sizes):
    specs = [(nx, ny, 1.5 + 0.3 * i / len(sizes)) for i, (nx, ny) in enumerate(sizes)]
    b = Batch(specs)
    fields = [inputs.random_fields(nx, ny, seed=i) for i, (nx, ny, _) in enumerate(specs)]
    for i, f in enumerate(fields):
        b.init(i, *f)
    for n in (3, 17, 2, 9):
        b.step(n)
    for i, (nx, ny, om) in enumerate(specs):
        if i % 9 and i < len(specs) - 3:
            continue
        lat = Lattice(2, nx, ny, omega=om, storage="f32").init(*fields[i])
        for _ in range(31):
            lat.step(1)
        assert torch.equal(b.buffer(i), lat.f), (nx, ny)
    b.close()


# strips of three, up to 48 sizes and more: closed strips with one, two and four
# chunks side by side, several strips, ragged rows; pairs for two and four steps left
@pytest.mark.parametrize("sizes", [[(256, 250)] * 9 + [(448, 300)] * 4 + [(64, 700)] * 9 + [(31, 300), (700, 333)],
                                   [(200 + i, 250 + 3 * i) for i in range(50)]])
def test_three_fused_batch_steps_equal_single_lattices(sizes):
    specs = [(nx, ny, 1.5 + 0.3 * i / len(sizes)) for i, (nx, ny) in enumerate(sizes)]
    b = Batch(specs)
    fields = [inputs.random_fields(nx, ny, seed=i) for i, (nx, ny, _) in enumerate(specs)]
    for i, f in enumerate(fields):
        b.init(i, *f)
    for n in (3, 4, 7, 8, 1, 2):
        b.step(n)
    for i, (nx, ny, om) in enumerate(specs):
        if i % 7 and i < len(specs) - 2:
            continue
        lat = Lattice(2, nx, ny, omega=om, storage="f32").init(*fields[i])
        for _ in range(25):
            lat.step(1)
        assert torch.equal(b.buffer(i), lat.f), (nx, ny)
    b.close()


# D3Q125: a row of two copies of a periodic row keeps both copies, whether the rows
# are taken by waves or whole, and however they are stored (ragged, on half lines)
@pytest.mark.parametrize("nx", [100, 102, 104, 120, 125, 128, 129, 250])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_box_rows_side_by_side_equal_one(nx, storage):
    ny, nz = 4, 5
    g = torch.Generator().manual_seed(nx)
    fields = [c + a * torch.rand(nz, ny, nx, generator=g, dtype=torch.float64)
              for c, a in ((1.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.0, 0.02), (0.4, 0.01))]
    a, b = (Lattice3(n, ny, nz, omega=1.2, storage=storage) for n in (nx, 2 * nx))
    a.init(*fields)
    b.init(*(f.repeat(1, 1, 2) for f in fields))
    a.step(3)
    b.step(3)
    one, two = (lat.f.view(nz, ny, 125, lat.nx) for lat in (a, b))
    assert torch.equal(two, one.repeat(1, 1, 1, 2))


def test_sums_of_threads_and_streams_do_not_mix():
    """Calls that ask for sums share one scratch while it is free: threads on
    streams of their own get their own lattice's sums."""
    import threading
    n, steps = 4, 12
    lats = [[Lattice(2, 200 + 60 * i, 90, omega=1.7, storage="f64").init(
        *inputs.random_fields(200 + 60 * i, 90, seed=i)) for _ in range(2)] for i in range(n)]
    want = [[b.step(1, sums=True) for _ in range(steps)] for _, b in lats]
    torch.cuda.synchronize()
    got = [None] * n

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            got[i] = [lats[i][0].step(1, sums=True) for _ in range(steps)]

    threads = [threading.Thread(target=work, args=(i,)) for i in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == want
