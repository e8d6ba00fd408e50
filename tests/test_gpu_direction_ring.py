"""Low-precision CG adds the search directions of a round of 1, 2, 4 or 8
iterations to the solution together (the longest that divides check_every).
Truncated solves follow the same iterates whatever the cadence of their
checks, so their solutions must be bit-identical for every round length: cut
off inside a round, at its end, and run until the right-hand sides stop one
after the other and some iterate again.  A batch must follow its single solves
through incomplete rounds as well."""
import numpy as np
import pytest

import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402


def sources(L, n):
    # random, smooth and point-like: different iteration counts
    b = S.random_spinor(L, 71, n)
    if n > 1:
        b[1] = np.roll(b[0], 1, axis=-1) + 3.0
    if n > 2:
        b[2] = 0
        b[2].reshape(-1)[5] = 1.0
    return torch.from_numpy(np.ascontiguousarray(b)).to("cuda:0")


def context(L, seed):
    ctx = P.Context(L, 0.130, 0.01)
    ctx.set_gauge(torch.from_numpy(S.gauge_links(L, 0.3, seed)).to("cuda:0"))
    return ctx


@pytest.mark.parametrize("prec", ["F32", "F16", "BF16"])
@pytest.mark.parametrize("maxiter,tol", [(5, 1e-12), (8, 1e-12), (13, 1e-12), (4000, 3e-2)])
def test_rounds_are_bit_identical(prec, maxiter, tol):
    L, n = (6, 4, 2, 6), 3
    ctx = context(L, 72)
    b = sources(L, n)
    got = {}
    for every in (1, 2, 3, 4, 6, 8, 16):
        x = torch.zeros_like(b)
        p = P.solve_params(tol=tol, solver=P.TM_CG_LOW, inner_prec=getattr(P, "TM_" + prec), maxiter=maxiter,
                           check_every=every)
        _, st = ctx.solve(x, b, n, p, allow_noconv=True)
        torch.cuda.synchronize()
        got[every] = (x.cpu().numpy(), [q.iters for q in st])
    for every, (x, it) in got.items():
        assert it == got[1][1], (every, it, got[1][1])
        assert np.array_equal(x, got[1][0]), every
    ctx.close()


@pytest.mark.parametrize("solver,maxiter", [("LOW", 13), ("MIXED", 21), ("MIXED", 4000)])
def test_batch_rounds(solver, maxiter):
    lats, nrhs = [(6, 4, 2, 6), (4, 4, 4, 8)], [3, 2]
    ctxs = [context(L, 73 + k) for k, L in enumerate(lats)]
    bs = [sources(L, n) for L, n in zip(lats, nrhs)]
    p = P.solve_params(tol=1e-9, solver=getattr(P, "TM_CG_" + solver), inner_prec=P.TM_F16, maxiter=maxiter)
    want = []
    for c, b, n in zip(ctxs, bs, nrhs):
        x = torch.zeros_like(b)
        c.solve(x, b, n, p, allow_noconv=True)
        want.append(x)
    batch = P.Batch(ctxs)
    xs = [torch.zeros_like(b) for b in bs]
    batch.solve(xs, bs, nrhs, p, allow_noconv=True)
    torch.cuda.synchronize()
    for x, w in zip(xs, want):
        assert torch.equal(x, w)
    batch.close()
    for c in ctxs:
        c.close()
