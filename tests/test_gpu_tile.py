"""The tile pass (several steps per launch, the automatic mode's way to step)
is bitwise the single sweeps it replaces: every storage type and boundary
combination, sizes at which each tile shape is chosen and around the columns
and rows a tile stores, remainders of every length, the models with and
without a compiled fast path, and the history of recorded steps."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1411_7051_amd import Batch, Lattice, inputs  # noqa: E402

STORAGES = ("f32", "f16", "bf16")


def drive(bcx):
    if bcx == inputs.PRESSURE:
        return dict(bc_x=bcx, rho_in=1.01, rho_out=1.0, init=1)
    return dict(bc_x=bcx, gx=2e-5, gy=-1e-5)


def same(case, steps, storage="f32", **extra):
    params = dict(case.params, **extra)
    states = []
    for mode in ("single", "auto"):
        lat = Lattice(case.eps, case.k, case.kn0, storage=storage, pass_mode=mode, check_every=0,
                      **params)
        for n in steps:
            lat.step(n)
        states.append(lat.save_state())
        lat.close()
    return torch.equal(*states)


def medium(nx, ny, seed=1, **params):
    return inputs.random_medium(nx, ny, seed=seed, solid_frac=0.04, pore_frac=0.05, **params)


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("bcx", [inputs.PERIODIC, inputs.WALL, inputs.PRESSURE])
@pytest.mark.parametrize("bcy", [inputs.PERIODIC, inputs.WALL])
def test_tile_bitwise(storage, bcx, bcy):
    small = [(3, 1), (5, 2), (57, 3), (58, 9), (59, 10), (61, 11), (64, 32), (117, 23), (174, 5)]
    if bcx != inputs.PRESSURE:
        small += [(1, 1), (2, 3)]
    for nx, ny in small:
        assert same(medium(nx, ny, bc_y=bcy, **drive(bcx)), (7, 2, 1, 5), storage), (nx, ny)
    # the larger shapes: 12 and 16 waves, 3 to 5 steps, one and two rows a wave
    for nx, ny in ((200, 160), (256, 256), (384, 256), (509, 511), (1111, 1025)):
        assert same(medium(nx, ny, bc_y=bcy, **drive(bcx)), (11,), storage), (nx, ny)


@pytest.mark.parametrize("extra", [dict(f_eps=0.7), dict(correlation=1), dict(correlation=2),
                                   dict(slip_b=-0.5), dict(kn_local=0), dict(rho_ref=1.5),
                                   dict(gx=1e-5), dict(gy=-1e-5), dict(tau=1.3)])
def test_tile_models(extra):
    for nx, ny in ((130, 37), (1030, 1021)):
        for storage in ("f32", "f16"):
            case = medium(nx, ny, seed=2, bc_y=inputs.WALL, **drive(inputs.PRESSURE))
            assert same(case, (8,), storage, **extra), (nx, ny, storage)


@pytest.mark.parametrize("bcx,obj,storage", [(inputs.PRESSURE, "k_app", "f32"),
                                             (inputs.PRESSURE, "q_out", "f16"),
                                             (inputs.PERIODIC, "k_app", "bf16")])
def test_tile_recording(bcx, obj, storage):
    for nx, ny in ((70, 41), (300, 230)):
        case = medium(nx, ny, seed=3, **drive(bcx))
        out = []
        for mode in ("single", "auto"):
            lat = Lattice(case.eps, case.k, case.kn0, storage=storage, pass_mode=mode,
                          **case.params)
            out.append(lat.gradient(23, obj, ckpt_every=14, hist_len=9, wrt_kn0=True))
            lat.close()
        assert out[0][0] == out[1][0]
        assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][2], out[1][2])


BATCH_SIZES = [(33, 7), (300, 41), (59, 130), (130, 64), (3, 2), (517, 90)]


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("bcx,bcy", [(inputs.PRESSURE, inputs.PERIODIC),
                                     (inputs.PRESSURE, inputs.WALL),
                                     (inputs.PERIODIC, inputs.WALL),
                                     (inputs.WALL, inputs.PERIODIC)])
@pytest.mark.parametrize("graph", [0, 10, 14])
def test_batch_tile_bitwise(storage, bcx, bcy, graph):
    """Tile passes over a batch (remainders shorter than a whole pass, graph
    replays of odd and even numbers of launches) against single sweeps of
    each sample; with FP32 the samples' models differ."""
    cases = [medium(nx, ny, seed=10 + i, bc_y=bcy, **drive(bcx))
             for i, (nx, ny) in enumerate(BATCH_SIZES)]
    extra = [dict(rho_ref=1.0 + 0.5 * (i & 1)) if storage == "f32" else {} for i in range(6)]
    lats = [Lattice(c.eps, c.k, c.kn0, storage=storage, **dict(c.params, **e))
            for c, e in zip(cases, extra)]
    solo = [Lattice(c.eps, c.k, c.kn0, storage=storage, pass_mode="single", check_every=0,
                    **dict(c.params, **e)) for c, e in zip(cases, extra)]
    b = Batch(lats)
    b.set_launch(64, 2, 0, graph)
    for n in (1, 7, 29):
        b.step(n)
    for a, s in zip(lats, solo):
        s.step(37)
        assert torch.equal(a.save_state(), s.save_state())


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_batch_pressure_columns(storage):
    # more than 1024 tiles: from 64 columns on a sample's pressure columns are in one strip
    cases = [medium(nx, 3001, seed=nx, bc_y=inputs.WALL, **drive(inputs.PRESSURE))
             for nx in (3, 63, 64, 65, 84, 85, 108, 111, 112, 113, 140)]
    out = []
    for mode in ("single", "auto"):
        lats = [Lattice(c.eps, c.k, c.kn0, storage=storage, check_every=0, **c.params)
                for c in cases]
        b = Batch(lats)
        b.set_pass_mode(mode)
        b.step(9)
        b.step(4)
        out.append([lat.save_state() for lat in lats])
    for c, x, y in zip(cases, *out):
        assert torch.equal(x, y), c.eps.shape


def test_batch_tile_large_and_gradient():
    """Two rows a wave (a batch of 2^21 nodes), and a batched gradient whose
    recomputing passes are tile passes."""
    cases = [medium(nx, ny, seed=20, **drive(inputs.PRESSURE))
             for nx, ny in ((1200, 900), (700, 1500))]
    lats = [Lattice(c.eps, c.k, c.kn0, storage="f16", **c.params) for c in cases]
    Batch(lats).step(13)
    for a, c in zip(lats, cases):
        s = Lattice(c.eps, c.k, c.kn0, storage="f16", pass_mode="single", **c.params)
        s.step(13)
        assert torch.equal(a.save_state(), s.save_state())
    cases = [medium(nx, ny, seed=30 + i, **drive(inputs.PRESSURE))
             for i, (nx, ny) in enumerate(BATCH_SIZES)]
    lats = [Lattice(c.eps, c.k, c.kn0, **c.params) for c in cases]
    J, g, gk = Batch(lats).gradient(23, ckpt_every=13, hist_len=6, wrt_kn0=True)
    for i, c in enumerate(cases):
        s = Lattice(c.eps, c.k, c.kn0, pass_mode="single", **c.params)
        Js, gs, gks = s.gradient(23, ckpt_every=13, hist_len=6, wrt_kn0=True)
        assert J[i] == Js and torch.equal(g[i], gs) and torch.equal(gk[i], gks)
