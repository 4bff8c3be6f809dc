"""Sampling of fe_profile inside the structured matrix-free CG, whose even launches move more than the odd ones:
an even stride k takes launches 0, k - 1, 2k, 3k - 1, ..., an odd one 0, k, 2k, ..., so both kinds are
timed equally often.  A solve of `it` iterations runs it + 1 launches, so the number of records tells which
launches were taken.  The assembled solve, whose launches are alike, keeps 0, k, 2k, ...
"""
import pytest

pytestmark = pytest.mark.gpu


def _count(launches, k, alternate):
    return sum(1 for b in range(launches + 1) if b * k - (b & 1 if alternate and k % 2 == 0 else 0) < launches)


@pytest.mark.parametrize("op", ["matfree", "csr"])
def test_even_strides_take_both_parities(op):
    import torch
    from paper_2604_22087_amd import fe
    n = 6
    P = fe.Problem(n, "f64")
    P.set_materials(torch.zeros(n ** 3, dtype=torch.uint8, device="cuda"), [fe.LINEAR], [(3.5, 0.35, 0, 0)])
    g = torch.Generator(device="cuda").manual_seed(1)
    b = torch.rand(P.n_dof, generator=g, dtype=torch.float64, device="cuda")
    P.set_dirichlet((b < 0.3).to(torch.uint8))
    kw, cls = dict(op=fe.OP_MATFREE), "matfree_apply"
    if op == "csr":
        kw, cls = dict(op=fe.OP_CSR, csr=(*P.csr_indices(), P.tangent_csr(b, apply_bc=True))), "csr_spmv"
    for k in (1, 2, 3, 4, 16):
        for it in (1, 2, 3, 4, 5, 8, 9, 16, 17, 18):
            print(f"[profile parity] op={op} k={k} it={it}", flush=True)
            P.profile(k)
            _, info = P.pcg(b, rtol=0.0, max_it=it, check=False, **kw)
            got = P.profile_read()[cls][0]
            P.profile(False)
            assert info.iterations == it
            assert got == _count(it + (op == "matfree"), k, op == "matfree")
