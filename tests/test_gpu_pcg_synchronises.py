"""fe_pcg synchronises its stream: at its return x is complete and nothing is left to run, after odd and even
numbers of iterations (the structured solve completes x in a launch of its own after an odd one).  The
mesh is large enough (6.4 M dofs) that a pass over x outlasts the return to the caller.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("iters", [1, 2, 3])
def test_stream_is_idle_when_pcg_returns(iters):
    import torch
    from paper_2604_22087_amd import fe
    print(f"[pcg synchronises] iters={iters}", flush=True)
    n = 128
    P = fe.Problem(n, "f64")
    P.set_materials(torch.zeros(n ** 3, dtype=torch.uint8, device="cuda"), [fe.LINEAR], [(3.5, 0.35, 0, 0)])
    b, x = torch.ones(P.n_dof, dtype=torch.float64, device="cuda"), P.vector()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(4):
            _, info = P.pcg(b, x, op=fe.OP_MATFREE, rtol=0.0, max_it=iters, check=False)
            idle = side.query()
            assert info.iterations == iters and idle
