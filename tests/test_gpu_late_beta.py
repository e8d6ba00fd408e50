"""The beta step of a CG iteration runs in a launch of its own or, with few partial
sums, inside the vector update and beside the next iteration.  Right-hand sides of
one call follow their single solves bit for bit in either form: 12^3 x 24, where one
right-hand side takes the second form, and the 16 of plain and truncated solves and
the 32 with reliable updates the first."""
import numpy as np
import pytest

import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402


@pytest.mark.parametrize("solver,n,tol", [("F64", 16, 1e-6), ("LOW", 16, 1e-2), ("MIXED", 32, 1e-7)])
def test_many_right_hand_sides_follow_their_single_solves(solver, n, tol):
    L = (12, 12, 12, 24)
    ctx = P.Context(L, 0.124, 0.01)
    ctx.set_gauge(torch.from_numpy(S.gauge_links(L, 0.3, 61)).to("cuda:0"))
    g = torch.Generator(device="cuda:0")
    g.manual_seed(62)
    b = torch.randn((n, ctx.V, 4, 3), dtype=torch.complex128, device="cuda:0", generator=g)
    if solver == "MIXED":
        b[:] = b[0].clone()  # reliable updates are common to the right-hand sides
    else:
        b[1] = 0
        b[1, 17, 2, 1] = 1.0  # another iteration count than the random ones
    x = torch.zeros_like(b)
    p = P.solve_params(tol=tol, solver=getattr(P, "TM_CG_" + solver), inner_prec=P.TM_F16)
    _, st = ctx.solve(x, b, n, p)
    for r in (0, 1, n - 1):
        one = torch.zeros_like(b[:1])
        _, s1 = ctx.solve(one, b[r:r + 1].contiguous(), 1, p)
        torch.cuda.synchronize()
        assert torch.equal(x[r:r + 1], one), r
        assert st[r].iters == s1[0].iters, r
    ctx.close()
