"""Where fe_pcg polls its solve (chunks of 8, 16, 32, ... iterations, cut at max_it and at the predicted
stop): iteration counts on both sides of every chunk edge, and the residual norm of the returned x against
the reported one, for the structured, the general-mesh and the assembled solve.

The recurrence residual and b - A x agree to about iterations * 1e-16 in FP64 while the
residual is far from that level (few iterations, rtol 1e-4); the bar is 1e-6 relative.
"""
import numpy as np
import pytest

from paper_2604_22087_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["grid", "mesh", "csr"])
def test_iteration_counts_around_the_polls(form):
    import torch
    from paper_2604_22087_amd import fe
    n = 7
    t = lambda a: torch.tensor(np.asarray(a), device="cuda")  # noqa: E731
    if form == "mesh":
        i = np.arange(n + 1)
        kk, jj, ii = np.meshgrid(i, i, i, indexing="ij")
        xyz = np.stack([ii.ravel(), jj.ravel(), kk.ravel()], axis=1) / n
        c, b, a = np.meshgrid(np.arange(n), np.arange(n), np.arange(n), indexing="ij")
        base = np.stack([a.ravel(), b.ravel(), c.ravel()], axis=1)
        off = np.array([(0, 0, 0), (1, 0, 0), (1, 1, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (1, 1, 1), (0, 1, 1)])
        corner = base[:, None, :] + off[None]
        P = fe.Problem(precision="f64", mesh=(xyz, corner[..., 0] + (n + 1) * (corner[..., 1] + (n + 1) * corner[..., 2])))
    else:
        P = fe.Problem(n, "f64")
    P.set_materials(t(inputs.sphere_phase(n)), [fe.LINEAR, fe.LINEAR], [(3.5, 0.35, 0, 0), (70.0, 0.22, 0, 0)])
    mask = inputs.boundary_dof_mask(n)
    P.set_dirichlet(t(mask))
    b = t(np.random.default_rng(2).normal(size=P.n_dof) * (1 - mask))
    kw = dict(op=fe.OP_MATFREE)
    if form == "csr":
        kw = dict(op=fe.OP_CSR, csr=(*P.csr_indices(), P.tangent_csr(b, apply_bc=True)))

    def relres(x):
        return float((b - P.apply_matfree(x, apply_bc=True)).norm() / b.norm())

    for it in (0, 1, 7, 8, 9, 10, 23, 24, 25, 26):
        print(f"[cg polls] form={form} max_it={it}", flush=True)
        x, info = P.pcg(b, rtol=1e-14, max_it=it, check=False, **kw)
        assert info.iterations == it and info.status != 0
        assert info.relres == pytest.approx(relres(x), rel=1e-6)
    for rtol in (0.3, 1e-1, 1e-2, 1e-4):
        x, info = P.pcg(b, rtol=rtol, max_it=1000, **kw)
        assert info.status == 0 and info.relres <= rtol
        assert info.relres == pytest.approx(relres(x), rel=1e-6)
        _, short = P.pcg(b, rtol=rtol, max_it=info.iterations - 1, check=False, **kw)
        assert short.iterations == info.iterations - 1 and short.status != 0
