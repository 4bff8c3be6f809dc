"""The point-wise reverse sweep of fe_vjp_path on sizes around the element bricks (one element, a brick
edge, ragged) against central differences of the library's own FP64 residual and return map: the
contraction c.R + mu.h is differentiated along random directions in the starting state, the
modulus scale and (its history part) the displacement.

Central differences with a step d have relative error about d^2 |f'''| / 6 + 1e-16 |f| / (d |f'|);
with steps of 1e-6 in strain units and fields of order 1e-2 both terms stay below 1e-7, except at the
few points whose trial state sits within a step of yield; the bar is 1e-5.
"""
import numpy as np
import pytest

from helpers import PHASES_J2_FIBER, lib_materials
from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4, 17])
def test_path_adjoint_directional(n):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[path adjoint point] n={n}", flush=True)
    rng = np.random.default_rng(n)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")  # noqa: E731
    ne = n ** 3
    phase = torch.tensor(((rng.random(ne) < 0.3) & (n > 1)).astype(np.uint8), device="cuda")
    models, params = lib_materials(PHASES_J2_FIBER)
    P = fe.Problem(n, "f64")
    scale = t(rng.uniform(0.8, 1.2, ne))
    idx = np.arange(n + 1) / n
    kk, jj, ii = np.meshgrid(idx, idx, idx, indexing="ij")
    u = np.stack([0.03 * ii.ravel(), -0.01 * jj.ravel(), 0 * kk.ravel()], axis=1).ravel()
    u = t(u + inputs.random_displacement(n, -0.006 / n, 0.006 / n, seed=4))
    j2 = (phase == 0).double().repeat(8 * 7)
    hist = t(rng.normal(scale=1e-3, size=56 * ne))
    hist[48 * ne:].abs_()
    hist *= j2
    c, mu = t(rng.normal(size=P.n_dof)), t(rng.normal(size=56 * ne))

    def value(u_, h_, s_, with_c=True):
        P.set_materials(phase, models, params, scale=s_)
        trial = P.state()
        r = P.residual(u_, h_, trial)
        return (float(c @ r) if with_c else 0.0) + float(mu @ trial)

    du = t(rng.normal(size=P.n_dof)) / n
    dh, ds = t(rng.normal(size=56 * ne)) * j2, t(rng.normal(size=ne))
    P.set_materials(phase, models, params, scale=scale)
    u_bar, s_bar = P.vector(), torch.zeros(ne, dtype=torch.float64, device="cuda")
    mu_out = P.vjp_path(u, hist, c, mu, None, u_bar, s_bar)
    d = 1e-6
    for got, fd in ((float(mu_out @ dh), (value(u, hist + d * dh, scale) - value(u, hist - d * dh, scale)) / (2 * d)),
                    (float(s_bar @ ds), (value(u, hist, scale + d * ds) - value(u, hist, scale - d * ds)) / (2 * d)),
                    (float(u_bar @ du), (value(u + d * du, hist, scale, False) - value(u - d * du, hist, scale, False)) / (2 * d))):
        assert got == pytest.approx(fd, rel=1e-5, abs=1e-9)
    # without cotangents of either kind the starting state's cotangent is the pass-through alone
    zero = P.vjp_path(u, hist, None, None)
    assert float(zero.abs().max()) == 0.0
