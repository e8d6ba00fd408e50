"""The ring of search directions of the low-precision solvers is optional memory.
With a limit on a context's workspace that the calls before it fit, a larger call
after a solve takes the ring back; where it does not fit, solves follow the same
iterates without one, alone and in a batch beside a lattice that has it."""
import pytest

import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402

DEV = "cuda:0"
MIXED = dict(tol=1e-7, solver=P.TM_CG_MIXED, inner_prec=P.TM_F16)


def free(b):
    x = torch.zeros_like(b)  # torch keeps the memory for the next solution
    torch.cuda.synchronize()
    del x
    return torch.cuda.mem_get_info()[0]


def context(L, seed, monkeypatch=None, limit=None):
    if limit is not None:
        monkeypatch.setenv("TM_WORKSPACE_LIMIT", str(limit))
    ctx = P.Context(L, 0.124, 0.01)
    if limit is not None:
        monkeypatch.delenv("TM_WORKSPACE_LIMIT")
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


def test_a_larger_call_takes_the_ring_back(monkeypatch):
    # the ring (264 MB) is more than the rounding of the measured use to pages
    L, n = (16, 16, 16, 32), 12
    b = sources(L, n, 51)
    gmres = dict(tol=1e-9, solver=P.TM_FGMRES, maxiter=3)
    ring = 7 * (b[0].numel() // 2) * 4 * n
    ctx = context(L, 50)  # also loads what the runtime loads at the first calls
    wantm, want = solve(ctx, b, **MIXED), solve(ctx, b, **gmres)
    ctx.close()
    ctx = context(L, 50)
    f0 = free(b)
    solve(ctx, b, check_every=1, **MIXED)  # no ring
    first = f0 - free(b)
    solve(ctx, b, **gmres)
    both = f0 - free(b)
    assert both > first + 8 * ring  # the second call is the larger one
    ctx.close()
    ctx = context(L, 50, monkeypatch, both)
    for _ in range(2):
        x, it = solve(ctx, b, **MIXED)
        assert torch.equal(x, wantm[0]) and it == wantm[1]
        x, it = solve(ctx, b, **gmres)
        assert torch.equal(x, want[0]) and it == want[1]
    ctx.close()


def test_solves_without_room_for_the_ring(monkeypatch):
    # one direction (75 MB) is more than the rounding of the measured use to pages
    L, n = (16, 16, 16, 32), 24
    b = sources(L, n, 53)
    ctx = context(L, 52)
    want = solve(ctx, b, **MIXED)
    ctx.close()
    ctx = context(L, 52)
    f0 = free(b)
    solve(ctx, b, check_every=1, **MIXED)
    used = f0 - free(b)
    ctx.close()
    ctx = context(L, 52, monkeypatch, used)
    x, it = solve(ctx, b, **MIXED)
    assert torch.equal(x, want[0]) and it == want[1]
    # beside a lattice with its ring: one length for both
    L2 = (8, 8, 8, 8)
    b2 = sources(L2, 2, 54)
    other = context(L2, 55)
    want2 = solve(other, b2, **MIXED)
    batch = P.Batch([ctx, other])
    xs = [torch.zeros_like(b), torch.zeros_like(b2)]
    batch.solve(xs, [b, b2], [n, 2], P.solve_params(**MIXED))
    torch.cuda.synchronize()
    assert torch.equal(xs[0], want[0]) and torch.equal(xs[1], want2[0])
    batch.close()
    other.close()
    ctx.close()
