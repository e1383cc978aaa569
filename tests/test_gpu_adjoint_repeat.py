"""A backward pass may be called again after one forward pass (first for ln k,
then with ln kn0): every call returns the gradients of the first bitwise, also
where a two-level plan rebuilds inner checkpoints in the slots of a segment
whose own the forward pass had kept."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1411_7051_amd import Batch, Lattice, _lib, inputs  # noqa: E402

STEPS, CKPT, HIST = 47, 13, 4  # four segments, the last one shorter


def medium(nx, ny, seed):
    return inputs.random_medium(nx, ny, seed=seed, solid_frac=0.04, pore_frac=0.05,
                                bc_x=inputs.PRESSURE, rho_in=1.01, rho_out=1.0, init=1)


@pytest.mark.parametrize("mode", ["auto", "single", "two_step"])
@pytest.mark.parametrize("segments", [0, 1, 2, 3])
def test_lattice(mode, segments):
    c = medium(90, 41, 5)
    lat = Lattice(c.eps, c.k, c.kn0, pass_mode=mode, **c.params)
    want = lat.gradient(STEPS, ckpt_every=CKPT, hist_len=HIST, wrt_kn0=True)
    lat.close()
    lat = Lattice(c.eps, c.k, c.kn0, pass_mode=mode, **c.params)
    nbytes = lat.adjoint_workspace_bytes(STEPS, CKPT, HIST)
    # room for the inner checkpoints of further segments
    nbytes += segments * -(-CKPT // HIST) * lat.state_bytes()
    ws = torch.empty(nbytes, dtype=torch.uint8, device=lat.device)
    J, ws = lat.adjoint_forward(STEPS, "k_app", CKPT, HIST, ws)
    assert J == want[0]
    assert torch.equal(lat.adjoint_backward(ws), want[1])
    for _ in range(2):
        g, gk = lat.adjoint_backward(ws, wrt_kn0=True)
        assert torch.equal(g, want[1]) and torch.equal(gk, want[2])


@pytest.mark.parametrize("mode", ["auto", "single", "two_step"])
def test_batch(mode):
    cases = [medium(nx, ny, nx) for nx, ny in ((70, 33), (33, 50), (130, 21))]
    lats = [Lattice(c.eps, c.k, c.kn0, **c.params) for c in cases]
    b = Batch(lats)
    b.set_pass_mode(mode)
    lib, n = _lib.load(), len(lats)
    nbytes = b.adjoint_workspace_bytes(STEPS, CKPT, HIST)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=b.device)
    J = np.empty(n)
    _lib.check(lib.lbk_batch_adjoint_forward(b._handle(), _lib.OBJECTIVE["k_app"], STEPS, CKPT,
                                             HIST, ws.data_ptr(), nbytes,
                                             J.ctypes.data_as(ctypes.c_void_p)))
    for _ in range(3):
        g = [torch.empty((lat.ny, lat.nx), device=b.device) for lat in lats]
        _lib.check(lib.lbk_batch_adjoint_backward(
            b._handle(), ws.data_ptr(), nbytes,
            (ctypes.c_void_p * n)(*[t.data_ptr() for t in g]), None))
        for c, gi, Ji in zip(cases, g, J):
            s = Lattice(c.eps, c.k, c.kn0, **c.params)
            want = s.gradient(STEPS, ckpt_every=CKPT, hist_len=HIST)
            assert Ji == want[0] and torch.equal(gi, want[1])
            s.close()
