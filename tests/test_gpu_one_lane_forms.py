"""Element kernels with one lane per element, at ragged sizes just past the rules that choose them (49..52 elements a
side for CG and the FP64 residual, 61 and 83 for K x, 37 and up for the VJP), against the two-lane form of the same
quantity: deterministic mode always runs that one (and a textbook CG).  The VJP is held against residuals whose
modulus scale selects random subsets of the elements: sum over the subset of out_e = lambda . R.

Bars: 1e-12 (FP64) and 1e-5 (FP32) normwise for element operations, as in the other parity tests.  CG in FP32: each
of the five steps puts an error of some 1e-6 (vectors in FP32, sums in FP64) into coefficients of order one, so x
agrees to a few 1e-5; the bar is 2e-4.
"""
import numpy as np
import pytest

from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}


def _problem(n, prec, law):
    import torch
    from paper_2604_22087_amd import fe
    rng = np.random.default_rng(n)
    P = fe.Problem(n, prec)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=P.dtype, device="cuda")  # noqa: E731
    phase = torch.tensor((rng.random(n ** 3) < 0.3).astype(np.uint8), device="cuda")
    first = {"linear": (fe.LINEAR, (3.5, 0.35, 0, 0)), "j2": (fe.J2, (3.5, 0.35, 0.05, 0.1)),
             "nh": (fe.NEOHOOKE, (2.6, 0.3, 0, 0))}[law]
    scale = t(rng.uniform(0.5, 2.0, n ** 3))
    P.set_materials(phase, [first[0], fe.LINEAR], [first[1], (70.0, 0.22, 0, 0)], scale=scale)
    P.set_dirichlet(torch.tensor(inputs.boundary_dof_mask(n), device="cuda"))
    i = np.arange(n + 1) / n
    kk, jj, ii = np.meshgrid(i, i, i, indexing="ij")
    u = np.stack([0.02 * ii.ravel(), -0.006 * jj.ravel(), 0 * kk.ravel()], axis=1).ravel()
    u = t(u + inputs.random_displacement(n, -0.006 / n, 0.006 / n, seed=4))
    return P, u, t(rng.normal(size=P.n_dof)), phase, t


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


def _both(P, f):
    a = f()
    P.set_deterministic(True)
    b = f()
    P.set_deterministic(False)
    return a, b


@pytest.mark.parametrize("n,prec,law", [(61, "f64", "linear"), (83, "f32", "linear"), (83, "f32", "nh")])
def test_operator(n, prec, law):
    print(f"[one lane K x] n={n} prec={prec} law={law}", flush=True)
    P, u, x, _, _ = _problem(n, prec, law)
    P.residual(u, store_tangent=True)
    for bc in (False, True):
        a, b = _both(P, lambda: P.apply_matfree(x, apply_bc=bc))
        assert _rel(a, b) <= TOL[prec]
    if prec == "f32":
        P.set_fp32_accumulation(True)
        a, b = _both(P, lambda: P.apply_matfree(x, apply_bc=True))
        assert _rel(a, b) <= 1e-5


@pytest.mark.parametrize("n", [49, 52])
def test_residual_fp64_linear(n):
    print(f"[one lane residual] n={n}", flush=True)
    P, u, _, _, _ = _problem(n, "f64", "linear")
    for bc in (False, True):
        a, b = _both(P, lambda: P.residual(u, apply_bc=bc))
        assert _rel(a, b) <= 1e-12
    a, b = _both(P, lambda: P.mean_stress(u))
    assert a == pytest.approx(b, rel=1e-11, abs=1e-13)


@pytest.mark.parametrize("law", ["linear", "j2", "nh"])
@pytest.mark.parametrize("n", [49, 50, 52])
def test_cg_fp32(n, law):
    from paper_2604_22087_amd import fe
    print(f"[one lane CG] n={n} law={law}", flush=True)
    P, u, x, _, t = _problem(n, "f32", law)
    P.residual(u, store_tangent=True)
    if law == "j2":
        total, plastic = P.linearization_stats()
        assert 0 < plastic < total
    b = x * t(1.0 - inputs.boundary_dof_mask(n))
    for pc in (fe.PC_JACOBI, fe.PC_BLOCK_JACOBI):
        P.set_preconditioner(pc)
        for acc32 in (False, True):
            P.set_fp32_accumulation(acc32)
            a, c = _both(P, lambda: P.pcg(b, op=fe.OP_MATFREE, rtol=0.0, max_it=5, check=False)[0])
            assert _rel(a, c) <= 2e-4


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,law", [(37, "linear"), (37, "nh"), (64, "linear")])
def test_vjp(n, law, prec):
    import torch
    print(f"[one lane VJP] n={n} law={law} prec={prec}", flush=True)
    P, u, x, phase, t = _problem(n, prec, law)
    out = P.vjp(u, x).double()
    from paper_2604_22087_amd import fe
    first = {"linear": (fe.LINEAR, (3.5, 0.35, 0, 0)), "nh": (fe.NEOHOOKE, (2.6, 0.3, 0, 0))}[law]
    P.set_dirichlet(None)
    P.set_deterministic(True)
    for seed in range(3):
        sel = t((np.random.default_rng(seed).random(n ** 3) < 0.3).astype(float))
        P.set_materials(phase, [first[0], fe.LINEAR], [first[1], (70.0, 0.22, 0, 0)], scale=sel)
        r = P.residual(u).double()
        got, ref = float((out * sel.double()).sum()), float(r @ x.double())
        size = float((r.abs() * x.double().abs()).sum())
        assert abs(got - ref) <= TOL[prec] * size
    assert bool(torch.isfinite(out).all())
