"""Batched gradients whose recomputing passes are tile passes over more than 1024
tiles: from there on a sample's pressure columns share a strip of tiles, which
then records the history of columns from both ends.  Bitwise the gradients of
each sample alone in single sweeps and steps."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1411_7051_amd import Batch, Lattice, inputs  # noqa: E402

# below and above the 64 columns from which a strip holds both ends, and around
# the widths of one, two and three strips
WIDTHS = (3, 63, 64, 65, 71, 72, 73, 84, 85, 108, 111, 112, 113, 128, 140, 169)


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bcy", [inputs.PERIODIC, inputs.WALL])
@pytest.mark.parametrize("extra", [{}, dict(rho_ref=1.5)])
def test_pressure_columns(storage, bcy, extra):
    cases = [inputs.random_medium(nx, 3001, seed=nx, solid_frac=0.04, pore_frac=0.05,
                                  bc_x=inputs.PRESSURE, bc_y=bcy, rho_in=1.01, rho_out=1.0, init=1)
             for nx in WIDTHS]
    lats = [Lattice(c.eps, c.k, c.kn0, storage=storage, **dict(c.params, **extra)) for c in cases]
    b = Batch(lats)
    K = b.tile_steps
    assert K > 0
    # more than 1024 tiles, whichever of the shapes of K steps is taken: 64 - 2 K
    # columns by at most 32 - 2 K rows
    assert sum(-(-nx // (64 - 2 * K)) for nx in WIDTHS) * (3001 // (32 - 2 * K)) > 1024
    J, g, gk = b.gradient(13, ckpt_every=9, hist_len=5, wrt_kn0=True)
    for i, c in enumerate(cases):
        one = Lattice(c.eps, c.k, c.kn0, storage=storage, pass_mode="single",
                      **dict(c.params, **extra))
        Js, gs, gks = one.gradient(13, ckpt_every=9, hist_len=5, wrt_kn0=True)
        assert J[i] == Js, c.eps.shape
        assert torch.equal(g[i], gs) and torch.equal(gk[i], gks), c.eps.shape
        assert torch.equal(lats[i].save_state(), one.save_state()), c.eps.shape
        one.close()
