"""Matrix-free solves on a general mesh run on element forces gathered by node (21 nodes per wave, 32
elements per workgroup): meshes of one element up to a few workgroups, nonzero values on constrained
dofs, point and node-block Jacobi CG, BiCGStab and GMRES, against the FP64 oracle's CG.

Solves to 1e-13 (FP64) and 1e-6 (FP32) are compared to 1e-8 and 1e-4, as the other solver tests do.
"""
import numpy as np
import pytest

from helpers import PHASES_CONFIG1, lib_materials, oracle_phases, rel_err
from oracle import solver
from oracle.rve import RVE
from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 2, 3, 7])
def test_general_cg(n, prec):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[general cg] n={n} prec={prec}", flush=True)
    coords, conn = inputs.distorted_cube_mesh(n, amplitude=0.2, seed=5)
    phase = (np.random.default_rng(1).random(len(conn)) < 0.4).astype(np.uint8)
    rve = RVE(None, phase, oracle_phases(PHASES_CONFIG1), mesh=(coords, conn))
    mask = (np.asarray(coords)[:, 0] < 1e-12).astype(np.uint8).repeat(3)  # one face held, the rest free
    _, k_e, _ = rve.element_residual_tangent(np.zeros(3 * len(coords)))
    b = np.random.default_rng(2).normal(size=3 * len(coords))
    ref, it_ref, status, _ = solver.pcg(lambda v: solver.matfree_apply(rve.conn, k_e, v, mask),
                                        solver.matfree_diagonal(rve.conn, k_e, rve.n_dof, mask), b, 1e-13, 20000)
    assert status == solver.OK
    P = fe.Problem(precision=prec, mesh=(coords, conn))
    models, params = lib_materials(PHASES_CONFIG1)
    P.set_materials(torch.tensor(phase, device="cuda"), models, params)
    P.set_dirichlet(torch.tensor(mask, device="cuda"))
    rtol, tol = (1e-13, 1e-8) if prec == "f64" else (1e-6, 1e-4)
    bt = torch.tensor(b, dtype=P.dtype, device="cuda")
    for pc in (fe.PC_JACOBI, fe.PC_BLOCK_JACOBI):
        P.set_preconditioner(pc)
        x, res = P.pcg(bt, op=fe.OP_MATFREE, rtol=rtol)
        assert rel_err(x.double().cpu().numpy(), ref) <= tol
        if pc == fe.PC_JACOBI and prec == "f64":
            assert abs(res.iterations - it_ref) <= max(3, it_ref // 50)
        x2, _ = P.pcg(bt, op=fe.OP_MATFREE, rtol=rtol, max_it=3, check=False)  # stops at the limit
        assert bool(torch.isfinite(x2).all())
    if prec == "f64":
        for kind in (fe.SOLVER_BICGSTAB, fe.SOLVER_GMRES):
            x, _ = P.pcg(bt, op=fe.OP_MATFREE, rtol=rtol, solver=kind, restart=60)
            assert rel_err(x.cpu().numpy(), ref) <= tol
