"""CSR values on both sides of the tile rule (18^3 elements and more go by tiles of 4 x 4 x 2 nodes) and on ragged tiles:
column by column against the matrix-free operator of the same linearisation, whose kernels form no
matrix.  The matrix times a vector is compared at 1e-12 (FP64) and 1e-5 (FP32) as in the other operator
tests, on vectors that meet every row; symmetry and the rows of constrained dofs exactly.
"""
import numpy as np
import pytest

from helpers import PHASES_CONFIG1, PHASES_J2_FIBER, lib_materials, rel_err
from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu

LAWS = {"linear": PHASES_CONFIG1, "j2": PHASES_J2_FIBER,
        "nh": [("neohooke", 10.0, 0.3), ("linear", 50.0, 0.25)]}


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("law", ["linear", "j2", "nh"])
@pytest.mark.parametrize("n", [1, 3, 17, 18, 21, 26])
def test_rows_match_operator(n, law, prec):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[tangent tiles] n={n} law={law} prec={prec}", flush=True)
    P = fe.Problem(n, prec)
    rng = np.random.default_rng(n)
    ne = n ** 3
    phase = torch.tensor((rng.random(ne) < 0.3).astype(np.uint8), device="cuda")
    models, params = lib_materials(LAWS[law])
    t = lambda a: torch.tensor(a, dtype=P.dtype, device="cuda")  # noqa: E731
    P.set_materials(phase, models, params, t(rng.uniform(0.8, 1.2, ne)))
    idx = np.arange(n + 1) / n
    kk, jj, ii = np.meshgrid(idx, idx, idx, indexing="ij")
    # half the cube strained past yield, half elastic: whole elements in closed form and point by point
    u = np.stack([0.03 * np.maximum(ii - 0.5, 0).ravel(), 0 * jj.ravel(), 0 * kk.ravel()], axis=1).ravel()
    u = t(u + inputs.random_displacement(n, -1e-4 / n, 1e-4 / n, seed=4))
    mask = (rng.random(P.n_dof) < 0.05).astype(np.uint8)
    P.set_dirichlet(torch.tensor(mask, device="cuda"))
    row_ptr, col_idx = P.csr_indices()
    tol = 1e-12 if prec == "f64" else 1e-5
    for bc in (False, True):
        vals = P.tangent_csr(u, apply_bc=bc).double()
        A = torch.sparse_csr_tensor(row_ptr.long(), col_idx.long(), vals, (P.n_dof, P.n_dof))
        for seed in range(2):
            x = t(np.random.default_rng(seed).normal(size=P.n_dof))
            got = (A @ x.double()[:, None])[:, 0].cpu().numpy()
            assert rel_err(got, P.apply_matfree(x, apply_bc=bc).double().cpu().numpy()) <= tol
        rows = torch.repeat_interleave(torch.arange(P.n_dof, device="cuda"), (row_ptr[1:] - row_ptr[:-1]).long())
        cols = col_idx.long()
        order = torch.argsort(cols * P.n_dof + rows)  # the transpose's entries in this pattern's order
        assert rel_err(vals[order].cpu().numpy(), vals.cpu().numpy()) <= tol
        if bc:
            held = torch.tensor(mask, device="cuda").bool()
            touch = held[rows] | held[cols]
            assert bool((vals[touch] == (rows == cols)[touch].double()).all())
