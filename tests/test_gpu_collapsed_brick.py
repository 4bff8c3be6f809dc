"""General meshes with collapsed bricks (wedges: two local nodes of an element share one node): the CSR
values, the operator and the matrix-free solve, whose element forces are gathered by node, against a
dense assembly of the FP64 oracle's element Jacobians.  Bars as for the other general-mesh tests:
1e-12 (FP64) and 1e-5 (FP32) for operators, 1e-8 and 1e-4 for solves.
"""
import numpy as np
import pytest

from helpers import PHASES_CONFIG1, lib_materials, oracle_phases, rel_err
from oracle.rve import RVE
from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu


def _wedge_mesh(n):
    """The n^3 mesh whose element column at x = y = 0 has its nodes (0, 0, k) merged into (1, 0, k)."""
    coords, conn = inputs.distorted_cube_mesh(n, amplitude=0.1, seed=3, permute=False)
    m = n + 1
    to = np.arange(len(coords))
    to[np.arange(m) * m * m] += 1
    keep = np.unique(to)
    new = np.full(len(coords), -1)
    new[keep] = np.random.default_rng(5).permutation(len(keep))
    out = np.empty((len(keep), 3))
    out[new[keep]] = coords[keep]
    return out, new[to[conn]]


def _fan_mesh(m, layers):
    """m wedges around the z axis in each of `layers` layers: an axis node is in up to 2 m elements,
    twice in each, and the assembly's rows of more than 8 incidences are read in place."""
    ang = 2 * np.pi * np.arange(m) / m
    ring = np.stack([np.cos(ang), np.sin(ang)], axis=1)
    coords = [np.array([[0, 0, z]] + [[x, y, z] for x, y in ring], dtype=float) for z in np.linspace(0, 1, layers + 1)]
    conn = []
    for k in range(layers):
        for i in range(m):
            bot = [0, 1 + i, 1 + (i + 1) % m, 0]
            conn.append([k * (m + 1) + v for v in bot] + [(k + 1) * (m + 1) + v for v in bot])
    return np.concatenate(coords), np.array(conn)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [2, 3, 5, 12])
def test_collapsed_bricks(n, prec):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[collapsed brick] n={n} prec={prec}", flush=True)
    coords, conn = _wedge_mesh(n) if n <= 3 else _fan_mesh(n, 2)
    assert any(len(set(c)) < 8 for c in conn.tolist())
    nd = 3 * len(coords)
    rng = np.random.default_rng(n)
    phase = (rng.random(len(conn)) < 0.4).astype(np.uint8)
    rve = RVE(None, phase, oracle_phases(PHASES_CONFIG1), mesh=(coords, conn))
    _, k_e, _ = rve.element_residual_tangent(np.zeros(nd))
    dofs = (3 * conn[:, :, None] + np.arange(3)).reshape(len(conn), 24)
    K = np.zeros((nd, nd))
    np.add.at(K, (dofs[:, :, None], dofs[:, None, :]), np.asarray(k_e).reshape(len(conn), 24, 24))
    mask = (coords[:, 2] < 1e-12).astype(np.uint8).repeat(3)
    P = fe.Problem(precision=prec, mesh=(coords, conn))
    models, params = lib_materials(PHASES_CONFIG1)
    P.set_materials(torch.tensor(phase, device="cuda"), models, params)
    tol, stol, rtol = (1e-12, 1e-8, 1e-13) if prec == "f64" else (1e-5, 1e-4, 1e-6)
    x = rng.normal(size=nd)
    xt = torch.tensor(x, dtype=P.dtype, device="cuda")
    assert rel_err(P.apply_matfree(xt).double().cpu().numpy(), K @ x) <= tol
    row_ptr, col_idx = P.csr_indices()
    vals = P.tangent_csr(P.vector())
    got = torch.sparse_csr_tensor(row_ptr.long(), col_idx.long(), vals.double(), (nd, nd)).to_dense().cpu().numpy()
    assert rel_err(got, K) <= tol
    P.set_dirichlet(torch.tensor(mask, device="cuda"))
    held = mask.astype(bool)
    Kb = K.copy()
    Kb[held, :] = 0
    Kb[:, held] = 0
    Kb[held, held] = 1
    ref = np.linalg.solve(Kb, x)
    sol, _ = P.pcg(xt, op=fe.OP_MATFREE, rtol=rtol)
    assert rel_err(sol.double().cpu().numpy(), ref) <= stol
    if prec == "f64":
        sol, _ = P.pcg(xt, op=fe.OP_MATFREE, rtol=rtol, solver=fe.SOLVER_BICGSTAB)
        assert rel_err(sol.cpu().numpy(), ref) <= stol
