"""Rounding of the momentum-resolved contractions against sums in 80 bits: the 2-norm
of the error over that of the result is no larger than with site-by-site
derivatives and one chain per Fourier sum, whose figures on these inputs, rounded up
to two digits, are the bars (local and derivative insertions of the standard and
one-end estimators, in 1e-16)."""
import numpy as np
import pytest

import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CL, LD = np.clongdouble, np.longdouble
EPS = 0.0123
# lattice, right-hand sides, |n|^2 <=, bars
CASES = [((12, 12, 14, 8), 1, 1, ((4.1, 3.8), (2.5, 3.8))),
         ((16, 12, 10, 6), 4, 2, ((4.5, 4.5), (2.0, 4.5)))]


def gammas():
    g = np.zeros((4, 4, 4), complex)
    g[0][0, 3] = g[0][1, 2] = -1j
    g[1][0, 3] = g[1][3, 0] = -1
    g[1][1, 2] = g[1][2, 1] = 1
    g[2][0, 2], g[2][1, 3] = -1j, 1j
    g[3][0, 2] = g[3][1, 3] = 1
    g = [m if (m == m.conj().T).all() else m + m.conj().T for m in g]
    out = []
    for n in range(16):
        m = np.eye(4, dtype=complex)
        for mu in range(4):
            if n >> mu & 1:
                m = m @ g[mu]
        out.append(m)
    return out


def loops80(L, U, eta, s, moms):
    """[estimator STD, one-end][momentum][80][Lt]."""
    shape = L[::-1]
    W = U.reshape(4, *shape, 3, 3).astype(CL)
    W[3, L[3] - 1] *= -1

    def apply(M, f):
        return (M[..., None, :, :] * f[..., None, :]).sum(-1)

    def nabla(f, mu):
        back = np.conj(np.swapaxes(np.roll(W[mu], 1, 3 - mu), -1, -2))
        return apply(W[mu], np.roll(f, -1, 3 - mu)) - apply(back, np.roll(f, 1, 3 - mu))

    def outer(v, w):  # [b][a]
        return (v[..., :, None, :] * w.conj()[..., None, :, :]).sum(-1)

    pi2, G = 2 * np.arctan2(LD(0), LD(-1)), gammas()
    g5 = np.diag([1, 1, -1, -1])
    out = np.zeros((2, len(moms), 80, L[3]), CL)
    for e, (left, coef) in enumerate(((eta, 1.0), (s, 2j * EPS))):
        C = np.zeros((5,) + shape + (4, 4), CL)
        for r in range(s.shape[0]):
            v, w = (f[r].reshape(*shape, 4, 3).astype(CL) for f in (s, left))
            C[0] += outer(v, w)
            for mu in range(4):
                C[1 + mu] += (outer(nabla(v, mu), w) - outer(v, nabla(w, mu))) / 4
        for m, p in enumerate(moms):
            D = C
            for d in (0, 1, 2):  # x, y, z: the last site axis first
                ph = np.exp(1j * (pi2 * LD(int(p[d])) / LD(L[d])) * np.arange(L[d]).astype(LD))
                D = (D * ph.reshape((1,) * (4 - d) + (-1, 1, 1))).sum(4 - d)
            for n in range(16):
                X = G[n] if e == 0 else g5 @ G[n]
                out[e, m, n::16] = CL(coef) * (X.T * D).sum((-1, -2))
    return out


def case(L, n):
    return S.gauge_links(L, 0.3, 141), S.random_spinor(L, 142, n), S.random_spinor(L, 143, n)


def errors(P, L, n, p2max):
    U, eta, s = case(L, n)
    ctx = P.Context(L, 0.124, EPS)
    ctx.set_gauge(torch.from_numpy(U).to("cuda:0"))
    got = ctx.contract_momentum(*(torch.from_numpy(f).to("cuda:0") for f in (eta, s)), n,
                                P.TM_EST_STD | P.TM_EST_ONE_END, p2max, 1, derivative=1)
    ctx.close()
    ref = loops80(L, U, eta, s, P.momenta(p2max))
    norm = lambda x: float(np.sqrt((np.abs(x) ** 2).sum()))
    return [[norm(got[e][:, k] - ref[e][:, k]) / norm(ref[e][:, k]) for k in (slice(0, 16), slice(16, 80))]
            for e in range(2)]


@pytest.mark.parametrize("L,n,p2max,bars", CASES)
def test_no_further_from_80_bits(L, n, p2max, bars):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_1309_2256_amd as P
    got = errors(P, L, n, p2max)
    for e in range(2):
        for k in range(2):
            assert got[e][k] <= 1e-16 * bars[e][k], (got, bars)
