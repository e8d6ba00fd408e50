"""The network's forward pass in FP32 is defined to the bit: transports, spin mixing
and gather are ascending chains of FP32 fused multiply-adds, on the matrix cores as
in scalar code.  The chain is restated here in numpy (product exact and sum rounded to
64 bits of mantissa before FP32, which double rounding could miss once in 2^40
additions) for half-lattices of less than a tile of 32 sites, ragged and of several
tiles."""
import numpy as np
import pytest

import oracle as O
import synth as S

torch = pytest.importorskip("torch")

LATS = [(4, 2, 2, 2), (6, 2, 4, 2), (6, 10, 2, 4)]
F, X = np.float32, np.longdouble


def fma(a, b, c):
    return (a.astype(X) * b.astype(X) + c.astype(X)).astype(F)


def cmac(acc, a, b):
    """acc += a b on (real, imaginary) pairs."""
    r = fma(-a[1], b[1], fma(a[0], b[0], acc[0]))
    return r, fma(a[1], b[0], fma(a[0], b[1], acc[1]))


def parts(z):
    return z.real.astype(F), z.imag.astype(F)


def forward(L, t_bc, U, A, psi):
    """N(psi) for the collapsed weights A [9][9][4][4]; fields [V][4][3]."""
    V = int(np.prod(L))
    grid = np.arange(V).reshape(L[::-1])
    t = np.arange(V) // (V // L[3])

    def transport(k, f):
        if k == 0:
            return f
        mu = (k - 1) & 3
        shift = -1 if k <= 4 else 1
        n = np.roll(grid, shift, axis=3 - mu).reshape(V)
        W = U[mu] if k <= 4 else U[mu][n].conj().transpose(0, 2, 1)
        if mu == 3:
            W = np.where((t == (L[3] - 1 if k <= 4 else 0))[:, None, None], t_bc * W, W)
        W = parts(W)
        out = [np.zeros((V, 4, 3), F), np.zeros((V, 4, 3), F)]
        for r in range(3):
            acc = (np.zeros((V, 4), F), np.zeros((V, 4), F))
            for c in range(3):
                acc = cmac(acc, [w[:, r, c][:, None] for w in W], [p[n, :, c] for p in f])
            out[0][:, :, r], out[1][:, :, r] = acc
        return out

    f, A = parts(psi), parts(A)
    g = [transport(k, f) for k in range(9)]
    out = None
    for k in range(9):
        u = [np.zeros((V, 4, 3), F), np.zeros((V, 4, 3), F)]
        for a in range(4):
            acc = (np.zeros((V, 3), F), np.zeros((V, 3), F))
            for kp in range(9):
                for b in range(4):
                    acc = cmac(acc, [np.full((V, 3), p[k, kp, a, b]) for p in A], [p[:, b] for p in g[kp]])
            u[0][:, a], u[1][:, a] = acc
        u = transport(k, u)
        out = u if out is None else [o + p for o, p in zip(out, u)]
    return out[0].astype(float) + 1j * out[1].astype(float)


def case(L):
    """Links, collapsed weights that the two layers give exactly, and a source."""
    rng = np.random.default_rng(84)
    A = (0.3 * (rng.standard_normal((9, 9, 4, 4)) + 1j * rng.standard_normal((9, 9, 4, 4)))).astype(np.complex64)
    W1 = np.zeros((9, 9, 4, 4), complex)
    for p in range(9):
        W1[p, p] = np.eye(4)
    return S.gauge_links(L, 0.3, 85), A, W1, A.astype(complex), S.random_spinor(L, 86, 1)


@pytest.mark.parametrize("L", LATS)
def test_restated_chain_is_the_network(L):
    U, A, W1, W2, psi = case(L)
    ref = O.ptc_forward(L, -1, U, W1, W2, psi[0])
    assert np.abs(forward(L, -1, U, A, psi[0]) - ref).max() <= 2e-5 * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("L", LATS)
def test_forward_bits(L):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_1309_2256_amd as P
    U, A, W1, W2, psi = case(L)
    ctx = P.Context(L, 0.124, 0.01)
    ctx.set_gauge(torch.from_numpy(U).to("cuda:0"))
    ctx.ptc_set_weights(W1, W2)
    d = torch.from_numpy(psi).to("cuda:0")
    out = torch.zeros_like(d)
    ctx.ptc_apply(out, d, 1)
    torch.cuda.synchronize()
    assert np.array_equal(out[0].cpu().numpy(), forward(L, -1, U, A, psi[0]))
    ctx.close()
