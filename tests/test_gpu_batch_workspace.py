"""A batched gradient asks for no more workspace than it always did: sizes and
budgets kept from earlier plans stay good."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1411_7051_amd import Batch, Lattice, _lib, inputs  # noqa: E402

# (steps, ckpt_every, hist_len) and the bytes asked for when single steps and
# two-step passes were the only ones
PLANS = [(30, 30, 30), (60, 20, 7), (100, 10, 10)]
SIZES = {1: [1204992, 1049344, 1450752], 3: [19833856, 17270528, 23881216],
         33: [30875904, 26887424, 37173504]}
SAMPLES = {1: [(64, 32)], 3: [(130, 64), (300, 41), (59, 130)],
           33: [(40 + i, 20) for i in range(33)]}


@pytest.mark.parametrize("n", [1, 3, 33])
@pytest.mark.parametrize("mode", ["auto", "single", "two_step"])
def test_workspace(n, mode):
    cases = [inputs.random_medium(nx, ny, seed=i, bc_x=inputs.PRESSURE, rho_in=1.01, rho_out=1.0,
                                  init=1) for i, (nx, ny) in enumerate(SAMPLES[n])]
    lats = [Lattice(c.eps, c.k, c.kn0, **c.params) for c in cases]
    b = Batch(lats)
    b.set_pass_mode(mode)
    lib = _lib.load()
    for (steps, ckpt, hist), before in zip(PLANS, SIZES[n]):
        assert b.adjoint_workspace_bytes(steps, ckpt, hist) <= before
        assert b.adjoint_plan(steps, ckpt, budget=before) >= hist
        start = [lat.save_state() for lat in lats]
        ws = torch.empty(before, dtype=torch.uint8, device=b.device)
        J = np.empty(n)
        _lib.check(lib.lbk_batch_adjoint_forward(
            b._handle(), _lib.OBJECTIVE["k_app"], steps, ckpt, hist, ws.data_ptr(), before,
            J.ctypes.data_as(ctypes.c_void_p)))
        g = [torch.empty((lat.ny, lat.nx), device=b.device) for lat in lats]
        _lib.check(lib.lbk_batch_adjoint_backward(
            b._handle(), ws.data_ptr(), before,
            (ctypes.c_void_p * n)(*[t.data_ptr() for t in g]), None))
        for i in range(0, n, 8):
            lats[i].load_state(start[i])
            want = lats[i].gradient(steps, ckpt_every=ckpt, hist_len=hist)
            assert J[i] == want[0] and torch.equal(g[i], want[1])
