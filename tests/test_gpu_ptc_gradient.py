"""Network gradient on the matrix cores: tiles of 32 half-sites per sample and
parity.  Half-lattices below, at and above a tile, ragged ones, and sample
counts that leave blocks without work or give them several tiles, against the
oracle's reverse-mode gradients (1e-4, the bar of the FP32 transports); the
loss also against the single samples' (the same FP32 values summed in FP64 in
another order, 1e-12)."""
import numpy as np
import pytest

import oracle as O
import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402


@pytest.mark.parametrize("L,n", [((2, 2, 2, 2), 1), ((4, 4, 2, 2), 3), ((6, 4, 2, 6), 2), ((12, 10, 14, 16), 3)])
def test_gradient_tiles(L, n):
    kappa, eps, nc = 0.124, 0.0123, 10
    U = S.gauge_links(L, 0.3, 61)
    ctx = P.Context(L, kappa, eps)
    ctx.set_gauge(torch.from_numpy(U).to("cuda:0"))
    rng = np.random.default_rng(62)
    W1, W2 = (0.3 * (rng.standard_normal((9, nc, 4, 4)) + 1j * rng.standard_normal((9, nc, 4, 4))) for _ in range(2))
    ctx.ptc_set_weights(W1, W2)
    r, e = S.random_spinor(L, 63, n), S.random_spinor(L, 64, n)
    dr, de = (torch.from_numpy(f).to("cuda:0") for f in (r, e))
    loss, G1, G2 = ctx.ptc_loss_grad(dr, de, n, nc)
    rl, R1, R2 = O.ptc_loss_grad(L, -1, U, W1, W2, list(r), list(e))
    assert abs(loss - rl) <= 1e-5 * rl
    for got, ref in ((G1, R1), (G2, R2)):
        assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    one = [ctx.ptc_loss_grad(dr[k:k + 1], de[k:k + 1], 1, nc)[0] for k in range(n)]
    assert abs(loss - sum(one) / n) <= 1e-12 * loss
    ctx.close()
