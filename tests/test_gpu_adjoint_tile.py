"""The reverse tile pass (several reverse steps per launch, the automatic mode's
way through a gradient) is bitwise the single reverse steps it replaces: both
gradients, every boundary combination, the models with and without a compiled
fast path, sizes for each of its tile shapes and around the columns that a
pressure outlet reaches, and remainders of every length."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1411_7051_amd import Lattice, inputs  # noqa: E402


def check(nx, ny, bcx, bcy=inputs.PERIODIC, steps=11, hist_len=11, kn=True, **extra):
    drive = (dict(rho_in=1.01, rho_out=1.0, init=1) if bcx == inputs.PRESSURE
             else dict(gx=2e-5, gy=-1e-5))
    case = inputs.random_medium(nx, ny, seed=nx + ny, solid_frac=0.04, pore_frac=0.05, bc_x=bcx,
                                bc_y=bcy, **drive)
    out = []
    for mode in ("single", "auto"):
        lat = Lattice(case.eps, case.k, case.kn0, pass_mode=mode, **dict(case.params, **extra))
        out.append(lat.gradient(steps, "k_app", ckpt_every=steps, hist_len=hist_len, wrt_kn0=kn))
        lat.close()
    assert out[0][0] == out[1][0], (nx, ny)
    for a, b in zip(out[0][1:], out[1][1:]):
        if a is not None:
            assert torch.equal(a, b), (nx, ny, int((a != b).sum()))


@pytest.mark.parametrize("bcx", [inputs.PERIODIC, inputs.WALL, inputs.PRESSURE])
@pytest.mark.parametrize("bcy", [inputs.PERIODIC, inputs.WALL])
@pytest.mark.parametrize("kn", [False, True])
def test_boundaries(bcx, bcy, kn):
    # tiles own 52, 56, 54 or 58 columns and 4, 8, 22 or 10 rows
    for nx, ny in ((3, 3), (52, 4), (53, 9), (105, 31), (64, 32)):
        check(nx, ny, bcx, bcy, kn=kn)


@pytest.mark.parametrize("nx", [*range(62, 67), *range(104, 114)])
def test_outlet_columns(nx):
    check(nx, 11, inputs.PRESSURE)


@pytest.mark.parametrize("nx,ny", [(384, 256), (500, 510), (1031, 517)])
@pytest.mark.parametrize("extra", [{}, dict(f_eps=0.7), dict(correlation=1),
                                   dict(correlation=2, gx=1e-6)])
def test_shapes_and_models(nx, ny, extra):
    check(nx, ny, inputs.PRESSURE, inputs.WALL, **extra)


@pytest.mark.parametrize("hist_len", range(1, 10))
def test_remainders(hist_len):
    check(70, 41, inputs.PRESSURE, steps=13, hist_len=hist_len)
