"""fe_vjp_path at elements without stiffness: a modulus scale of 0 (a void of a design field) or a phase with
E = 0.  The modulus-scale cotangent is finite there and, for the voids, equals the one-sided difference.

Up to a scale of 1e-3 the voids stay elastic (stresses below 1e-3 of the yield stress for strains of 1e-2),
so c.R is linear in their scale and the difference quotient is exact but for its rounding,
1e-16 |c.R| / (1e-3 |slope|) < 1e-10; the bar is 1e-8.
"""
import numpy as np
import pytest

from helpers import PHASES_J2_FIBER, lib_materials
from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 17])
def test_modulus_cotangent_of_void_elements(n):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[path adjoint void] n={n}", flush=True)
    rng = np.random.default_rng(n)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")  # noqa: E731
    ne = n ** 3
    phase_h = (rng.random(ne) < 0.2).astype(np.uint8)
    phase_h[rng.random(ne) < 0.1] = 2  # a J2 phase with E = 0
    models, params = lib_materials(PHASES_J2_FIBER)
    models, params = list(models) + [fe.J2], list(params) + [(0.0, 0.3, 0.05, 0.1)]
    phase = torch.tensor(phase_h, device="cuda")
    void = t((rng.random(ne) < 0.3).astype(np.float64))
    scale = t(rng.uniform(0.8, 1.2, ne)) * (1 - void)
    P = fe.Problem(n, "f64")
    idx = np.arange(n + 1) / n
    kk, jj, ii = np.meshgrid(idx, idx, idx, indexing="ij")
    u = np.stack([0.01 * ii.ravel(), -0.003 * jj.ravel(), 0 * kk.ravel()], axis=1).ravel()
    u = t(u + inputs.random_displacement(n, -0.002 / n, 0.002 / n, seed=4))
    hist, c = P.state(), t(rng.normal(size=P.n_dof))

    def value(s_):
        P.set_materials(phase, models, params, scale=s_)
        return float(c @ P.residual(u, hist))

    ds = void * t(rng.uniform(0.5, 1.0, ne))
    P.set_materials(phase, models, params, scale=scale)
    s_bar = torch.zeros(ne, dtype=torch.float64, device="cuda")
    mu_out = P.vjp_path(u, hist, c, t(rng.normal(size=56 * ne)), None, None, s_bar)
    assert bool(torch.isfinite(s_bar).all()) and bool(torch.isfinite(mu_out).all())
    d = 1e-3
    assert float(s_bar @ ds) == pytest.approx((value(scale + d * ds) - value(scale)) / d, rel=1e-8)
