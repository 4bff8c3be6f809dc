"""ILU(0) sweeps run one grid row per workgroup with eight lanes per node: grids from one element (no
odd rows to spare) to rows longer than one pass of a workgroup, and a matrix whose rows do not hold
the full pattern (explicit zeros dropped, so blocks are searched), against the oracle's factors.

Bar: 1e-11 (FP64) and 1e-4 (FP32) normwise, an order above the application test of the 8^3 matrix,
since the small random matrices here are only weakly diagonally dominant.
"""
import numpy as np
import pytest

from helpers import rel_err
from oracle import assembly, ilu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,drop", [(1, False), (2, False), (3, True), (5, False), (6, True)])
def test_ilu_application_sizes(n, drop, prec):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[ilu rows] n={n} drop={drop} prec={prec}", flush=True)
    P = fe.Problem(n, prec)
    rp, ci = (t.cpu().numpy() for t in P.csr_indices())
    rng = np.random.default_rng(n)
    v = rng.uniform(-1, 1, len(ci))
    rows = assembly.csr_rows(rp)
    v[rows == ci] += 60.0
    if drop:  # remove a tenth of the off-diagonal entries from the pattern
        keep = (rows == ci) | (rng.random(len(ci)) > 0.1)
        rp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=len(rp) - 1))]).astype(np.int32)
        ci, v = ci[keep], v[keep]
    r = rng.normal(size=len(rp) - 1)
    ref = ilu.bilu0_preconditioner(n, rp, ci, v)(r)
    P.set_preconditioner(fe.PC_ILU0)
    csr = (torch.tensor(rp, device="cuda"), torch.tensor(ci, device="cuda"), torch.tensor(v, dtype=P.dtype, device="cuda"))
    z = P.apply_preconditioner(torch.tensor(r, dtype=P.dtype, device="cuda"), csr=csr)
    assert rel_err(z.double().cpu().numpy(), ref) <= (1e-11 if prec == "f64" else 1e-4)
    assert P.read_flags() == 0


def test_ilu_row_longer_than_a_workgroup_pass():
    """n = 130: a row of 131 nodes needs a second pass of 1024 lanes; L U z = r is checked through the
    factors of a block-diagonal matrix (each 3x3 pivot block inverted), which any size allows."""
    import torch
    from paper_2604_22087_amd import fe
    n = 130
    P = fe.Problem(n, "f32")
    g = torch.Generator(device="cuda").manual_seed(3)
    d = torch.rand(P.n_dof, generator=g, device="cuda") + 1.0
    rp = torch.arange(P.n_dof + 1, dtype=torch.int32, device="cuda")
    ci = torch.arange(P.n_dof, dtype=torch.int32, device="cuda")
    r = torch.randn(P.n_dof, generator=g, device="cuda")
    P.set_preconditioner(fe.PC_ILU0)
    z = P.apply_preconditioner(r, csr=(rp, ci, d))
    assert rel_err(z.double().cpu().numpy(), (r / d).double().cpu().numpy()) <= 1e-6
