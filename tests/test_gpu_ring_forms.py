"""The ring of search directions where its forms differ: a zero source beside
others never iterates and leaves the other directions of the ring unwritten, which
the hops of its lane read; a batch follows its single solves bit for bit with every
ring length (1, 2, 4 and 8 iterations by the cadence of the checks), as a
persistent launch and as a graph of launches."""
import pytest

import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402

DEV = "cuda:0"
MIXED = dict(tol=1e-7, solver=P.TM_CG_MIXED, inner_prec=P.TM_F16)


def context(L, seed):
    ctx = P.Context(L, 0.124, 0.01)
    ctx.set_gauge(torch.from_numpy(S.gauge_links(L, 0.3, seed)).to(DEV))
    return ctx


def sources(L, n, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn((n, L[0] * L[1] * L[2] * L[3], 4, 3), dtype=torch.complex128, device=DEV, generator=g)


def solve(ctx, b, **kw):
    x = torch.zeros_like(b)
    _, st = ctx.solve(x, b, b.shape[0], P.solve_params(**kw), allow_noconv=True)
    torch.cuda.synchronize()
    return x, [q.iters for q in st]


@pytest.mark.parametrize("solver", ["LOW", "MIXED"])
@pytest.mark.parametrize("prec", ["F32", "F16", "BF16"])
def test_a_zero_source_beside_others(solver, prec):
    L, n = (6, 4, 2, 6), 3
    b = sources(L, n, 56)
    b[1] = 0
    kw = dict(tol=3e-2 if solver == "LOW" else 1e-7, solver=getattr(P, "TM_CG_" + solver),
              inner_prec=getattr(P, "TM_" + prec))
    ctx = context(L, 57)
    x, it = solve(ctx, b, **kw)
    one, it1 = solve(ctx, b[:1].contiguous(), **kw)
    assert it[1] == 0 and not x[1].any()
    assert torch.isfinite(torch.view_as_real(x)).all()
    if solver == "LOW":
        assert torch.equal(x[:1], one) and it[0] == it1[0]
    ctx.close()


@pytest.mark.parametrize("form", ["1", "0"])
@pytest.mark.parametrize("every", [1, 2, 4, 8, 12])
def test_batches_with_every_ring_length(every, form, monkeypatch):
    monkeypatch.setenv("TM_BATCH_PERSIST", form)
    lats, nrhs = [(6, 4, 2, 6), (4, 4, 4, 8)], [3, 2]
    ctxs = [context(L, 58 + k) for k, L in enumerate(lats)]
    bs = [sources(L, n, 60 + k) for k, (L, n) in enumerate(zip(lats, nrhs))]
    kw = dict(MIXED, check_every=every)
    want = [solve(c, b, **kw) for c, b in zip(ctxs, bs)]
    batch = P.Batch(ctxs)
    xs = [torch.zeros_like(b) for b in bs]
    _, st = batch.solve(xs, bs, nrhs, P.solve_params(**kw))
    torch.cuda.synchronize()
    for x, (w, it), q in zip(xs, want, st):
        assert torch.equal(x, w) and [s.iters for s in q] == it
    batch.close()
    for c in ctxs:
        c.close()
