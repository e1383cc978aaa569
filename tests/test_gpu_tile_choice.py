"""Which passes the automatic mode takes: tile passes but on very wide lattices
of a few rows, where a tile loads many times the rows it stores, and on mid-sized lattices
with the Forchheimer term, 16-bit storage and pressure columns."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1411_7051_amd import Batch, Lattice, inputs  # noqa: E402

PRESSURE = dict(bc_x=inputs.PRESSURE, rho_in=1.01, rho_out=1.0, init=1, check_every=0)


def fields(nx, ny, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = [torch.rand((ny, nx), generator=g, device="cuda") for _ in range(3)]
    return 0.2 + 0.5 * r[0], 10 ** (-4 + 3 * r[1]), 0.01 + 0.2 * r[2]


# either side of the rule, per pass that tile passes replace (single sweeps, two-
# and three-step passes), where the measured times differ by a tenth and more
@pytest.mark.parametrize("nx,ny,storage,tiles", [
    (32768, 1, "f32", True), (131072, 1, "f32", False), (524288, 1, "f32", False),
    (262144, 2, "f32", True), (524288, 2, "f32", False), (524288, 3, "f32", False),
    (524288, 5, "f32", True), (1048576, 3, "f32", False), (1048576, 5, "f32", False),
    (524288, 13, "f32", True), (32768, 1, "f16", True), (131072, 1, "f16", False),
    (65536, 2, "f16", True), (262144, 2, "f16", False), (262144, 3, "bf16", False),
    (524288, 6, "f16", True), (1048576, 4, "f16", False), (1048576, 8, "bf16", False),
    (1048576, 12, "f16", False), (524288, 24, "f16", True), (3, 524288, "f32", True),
    (64, 32768, "f16", True)])
def test_wide_lattices(nx, ny, storage, tiles):
    f = fields(nx, ny)
    lat = Lattice(*f, storage=storage, **PRESSURE)
    assert (lat.tile_steps > 0) == tiles
    one = Lattice(*f, storage=storage, pass_mode="single", **PRESSURE)
    assert one.tile_steps == 0
    assert torch.equal(lat.step(8).save_state(), one.step(8).save_state())


# with the Forchheimer term: mid-sized lattices, and wide ones
@pytest.mark.parametrize("nx,ny,storage,bcx,tiles", [
    (777, 333, "f16", inputs.PRESSURE, True), (512, 512, "f16", inputs.PRESSURE, False),
    (1024, 512, "bf16", inputs.PRESSURE, False), (700, 400, "f16", inputs.PRESSURE, False),
    (1024, 1024, "f16", inputs.PRESSURE, False), (1400, 1400, "bf16", inputs.PRESSURE, True),
    (1024, 512, "f32", inputs.PRESSURE, True), (1024, 512, "f16", inputs.WALL, True),
    (1024, 1024, "bf16", inputs.PERIODIC, True), (24576, 1, "f16", inputs.PRESSURE, True),
    (65536, 1, "f32", inputs.PRESSURE, False), (262144, 2, "f32", inputs.PRESSURE, False),
    (1048576, 7, "f16", inputs.PRESSURE, False)])
def test_forchheimer(nx, ny, storage, bcx, tiles):
    drive = PRESSURE if bcx == inputs.PRESSURE else dict(bc_x=bcx, gx=1e-6, check_every=0)
    f = fields(nx, ny)
    lat = Lattice(*f, storage=storage, f_eps=0.5, **drive)
    assert (lat.tile_steps > 0) == tiles
    one = Lattice(*f, storage=storage, f_eps=0.5, pass_mode="single", **drive)
    assert torch.equal(lat.step(8).save_state(), one.step(8).save_state())


@pytest.mark.parametrize("nx,ny", [(16384, 1), (65536, 1), (32768, 4), (131072, 4), (524288, 4),
                                   (262144, 5), (524288, 5), (524288, 6), (400000, 11)])
@pytest.mark.parametrize("extra", [{}, dict(f_eps=0.7)])
def test_reverse_steps_of_wide_lattices(nx, ny, extra):
    """Either side of the reverse passes' rule: the gradients are those of
    single steps bitwise, and a backward pass takes no longer than with single
    sweeps and steps (an eighth is left for noise; the tile passes took 1.3 to
    2.8 times as long on the widest lattices of one to four rows)."""
    f = fields(nx, ny)
    runs = {}
    for mode in ("single", "auto"):
        lat = Lattice(*f, pass_mode=mode, **PRESSURE, **extra)
        _, ws = lat.adjoint_forward(12, "k_app", 12, 12)
        runs[mode] = (lat, ws, *lat.adjoint_backward(ws, wrt_kn0=True), [])
    assert torch.equal(runs["single"][2], runs["auto"][2])
    assert torch.equal(runs["single"][3], runs["auto"][3])
    for _ in range(25):
        for lat, ws, _, _, ms in runs.values():
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            lat.adjoint_backward(ws)
            ev[1].record()
            torch.cuda.synchronize()
            ms.append(ev[0].elapsed_time(ev[1]))
    assert min(runs["auto"][4]) <= 1.125 * min(runs["single"][4])


@pytest.mark.parametrize("n,nx,ny,storage,f_eps,tiles", [
    (64, 4096, 1, "f32", 0.0, False), (64, 8192, 2, "f32", 0.0, False),
    (64, 8192, 3, "f16", 0.0, False), (64, 8192, 4, "f32", 0.0, True),
    (64, 2000, 8, "f16", 0.0, True), (256, 100, 8, "f32", 0.0, True),
    (64, 8192, 3, "f32", 0.5, False), (64, 16384, 8, "bf16", 0.5, False),
    (12, 150, 160, "f32", 0.5, False), (12, 150, 160, "f32", 0.0, True),
    (2, 512, 512, "f16", 0.5, False), (2, 512, 512, "f32", 0.5, True),
    (16, 300, 200, "bf16", 0.5, True), (3, 1000, 900, "f16", 0.5, True)])
def test_batches(n, nx, ny, storage, f_eps, tiles):
    fs = [fields(nx, ny, i) for i in range(n)]
    lats = [Lattice(*f, storage=storage, f_eps=f_eps, **PRESSURE) for f in fs]
    b = Batch(lats)
    assert (b.tile_steps > 0) == tiles
    b.step(7)
    for f, lat in list(zip(fs, lats))[::max(1, n // 4)]:
        one = Lattice(*f, storage=storage, f_eps=f_eps, pass_mode="single", **PRESSURE)
        assert torch.equal(lat.save_state(), one.step(7).save_state())


# the steps of a whole tile pass at sizes that select each of its shapes (8, 12
# and 16 waves of one or two rows); the tests of bitwise equality compare the
# automatic mode with single sweeps at these sizes, so this is what they test
SHAPES = [(3, 1, 3), (64, 32, 3), (117, 23, 3), (70, 41, 3), (130, 37, 3), (200, 160, 4),
          (384, 256, 4), (256, 256, 5), (300, 230, 5), (509, 511, 3), (777, 333, 3),
          (1024, 512, 5), (1030, 1021, 4), (1111, 1025, 5)]


@pytest.mark.parametrize("nx,ny,steps", SHAPES)
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_steps_of_a_pass(nx, ny, steps, storage):
    f = fields(nx, ny)
    assert Lattice(*f, storage=storage, **PRESSURE).tile_steps == steps
    for bcx in (inputs.PERIODIC, inputs.WALL):
        lat = Lattice(*f, storage=storage, bc_x=bcx, bc_y=inputs.WALL, gx=1e-6, f_eps=0.7)
        assert lat.tile_steps == steps
    for mode in ("single", "two_step", "three_step"):
        assert Lattice(*f, storage=storage, pass_mode=mode, **PRESSURE).tile_steps == 0
    assert Lattice(*f, storage=storage, band=8, **PRESSURE).tile_steps == 0


@pytest.mark.parametrize("sizes,steps", [
    ([(33, 7), (300, 41), (59, 130), (130, 64), (3, 2), (517, 90)], 4),
    ([(1200, 900), (700, 1500)], 4),
    ([(nx, 3001) for nx in (3, 63, 64, 65, 84, 85, 108, 111, 112, 113, 140)], 4)])
def test_steps_of_a_batch_pass(sizes, steps):
    b = Batch([Lattice(*fields(nx, ny), **PRESSURE) for nx, ny in sizes])
    assert b.tile_steps == steps
    for mode in ("single", "two_step"):
        b.set_pass_mode(mode)
        assert b.tile_steps == 0
    b.set_pass_mode("auto")
    assert b.tile_steps == steps
