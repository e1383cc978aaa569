"""Gradients at very large Knudsen numbers: the derivative of the correction factor
stays finite as far as the forward's own numbers do (Kn = 1e15)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1411_7051_amd import Lattice, inputs  # noqa: E402


@pytest.mark.parametrize("kn", [1e10, 2e13, 1e14, 5e14])
@pytest.mark.parametrize("extra", [{}, dict(kn_local=0), dict(f_eps=0.5), dict(correlation=1)])
def test_large_kn(kn, extra):
    """The permeability is chosen so that k f_c, and so the flow, is ordinary
    whatever Kn.  Against central differences of the FP64 oracle, within the
    bounds of the gradient tests: 1e-3 of the largest gradient."""
    c = inputs.random_medium(24, 9, seed=7, kn_range=(0.5, 2.0), k_range=(0.5, 5.0),
                             bc_x=inputs.PRESSURE, rho_in=1.02, rho_out=1.0, init=1)
    kn0 = (c.kn0.astype(np.float64) * kn).astype(np.float32)
    k = (c.k / ((1.358 * 5.0 if extra.get("correlation") != 1 else 4.0) * kn)).astype(np.float32)
    params = dict(c.params, **extra)
    out = []
    for mode in ("auto", "single", "two_step"):
        lat = Lattice(c.eps, k, kn0, pass_mode=mode, **params)
        J, g, gk = lat.gradient(15, "k_app", ckpt_every=8, hist_len=3, wrt_kn0=True)
        assert np.isfinite(J) and bool(g.isfinite().all()) and bool(gk.isfinite().all())
        out.append((g, gk))
    assert all(torch.equal(a, b) for o in out[1:] for a, b in zip(out[0], o))
    nodes = [(y, x) for y in (0, 4, 8) for x in (0, 5, 11, 17, 23)]
    for g, wrt in zip(out[0], ("k", "kn0")):
        g = g.double().cpu().numpy()
        fd = oracle.fd_gradient(c.eps, k, kn0, 15, nodes, "k_app", h=1e-4, wrt=wrt, **params)
        err = np.abs(np.array([g[n] for n in nodes]) - fd)
        assert err.max() <= 1e-3 * np.abs(g).max(), (wrt, err.max(), np.abs(g).max())
