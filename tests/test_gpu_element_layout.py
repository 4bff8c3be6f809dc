"""Edges of the element kernels' lane layout (two lanes per element, bricks of 16 x 4 x 4): a single
element, exactly one brick width, one short of it and ragged sizes just past it, for a J2 RVE with
plastic history -- residual, mean stress, masked operator, and the fused CG launch with both
point preconditioners, against the FP64 oracle.

Tolerances are those of the other parity tests of the same quantities (1e-12 / 1e-5 normwise for
element operations, 1e-8 for a solve to 1e-13).
"""
import numpy as np
import pytest

from helpers import PHASES_J2_FIBER, lib_materials, oracle_phases, rel_err, state_to_lib
from oracle import assembly, solver
from oracle.rve import RVE
from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 4, 15, 16, 19])
def test_element_layout_edges(n, prec):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[element layout] n={n} prec={prec}", flush=True)
    phase = (np.random.default_rng(3).random(n ** 3) < 0.3).astype(np.uint8) * (n > 1)
    rve = RVE(n, phase, oracle_phases(PHASES_J2_FIBER))
    amp = 0.012 / n
    u = rve.affine_lift(np.diag([0.03, -0.01, 0.0])) + inputs.random_displacement(n, -amp, amp, seed=7)
    rng = np.random.default_rng(11)
    st = rve.zero_state()
    ep = rng.normal(scale=2e-3, size=st["eps_p"].shape)
    ep[..., 2] = -ep[..., 0] - ep[..., 1]
    st["eps_p"] = ep * (rve.phase == 0)[:, None, None]
    st["alpha"] = rng.uniform(0, 2e-3, st["alpha"].shape) * (rve.phase == 0)[:, None]
    r_e, k_e, trial = rve.element_residual_tangent(u, st)
    R = assembly.assemble_vector(rve.conn, r_e, rve.n_dof)
    mask = inputs.boundary_dof_mask(n)

    P = fe.Problem(n, prec)
    models, params = lib_materials(PHASES_J2_FIBER)
    P.set_materials(torch.tensor(phase, dtype=torch.uint8, device="cuda"), models, params)
    t = lambda a: torch.tensor(np.asarray(a), dtype=P.dtype, device="cuda")  # noqa: E731
    npy = lambda a: a.detach().double().cpu().numpy()  # noqa: E731
    tol = 1e-12 if prec == "f64" else 1e-5
    s_in = t(state_to_lib(st["eps_p"], st["alpha"]))
    assert rel_err(npy(P.residual(t(u), s_in, P.state(), store_tangent=True)), R) <= tol
    assert rel_err(P.mean_stress(t(u), s_in), rve.mean_stress(trial["sigma_all"])) <= tol
    x = rng.normal(size=rve.n_dof)
    assert rel_err(npy(P.apply_matfree(t(x))), solver.matfree_apply(rve.conn, k_e, x)) <= tol
    P.set_dirichlet(torch.tensor(mask, device="cuda"))
    assert rel_err(npy(P.apply_matfree(t(x), apply_bc=True)), solver.matfree_apply(rve.conn, k_e, x, mask)) <= tol
    if prec == "f32" or n == 1:
        return
    b = rng.normal(size=rve.n_dof)
    ref, _, status, _ = solver.pcg(lambda v: solver.matfree_apply(rve.conn, k_e, v, mask),
                                   solver.matfree_diagonal(rve.conn, k_e, rve.n_dof, mask), b, 1e-13, 5000)
    assert status == solver.OK
    for pc in (fe.PC_JACOBI, fe.PC_BLOCK_JACOBI):
        P.set_preconditioner(pc)
        w, _ = P.pcg(t(b), op=fe.OP_MATFREE, rtol=1e-13)
        assert rel_err(npy(w), ref) <= 1e-8
