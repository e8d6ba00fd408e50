"""Spin mixing of the network in FP32 and BF16 on the matrix cores: tiles of 32
half-sites per right-hand side.  Half-lattices below, at and above a tile and
ragged ones, fewer and more tiles than resident blocks.  The FP32
products are ascending chains of FMAs, and a batch must be bit-identical to its single
fields; against the FP64 oracle 2e-5 (FP32 rounding over ~10^3 accumulated
products) and for BF16 operands 2e-2 (unit roundoff 4e-3 on every operand, of
random sign over the sum)."""
import numpy as np
import pytest

import oracle as O
import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402


@pytest.mark.parametrize("arith,bar", [(P.TM_F32, 2e-5), (P.TM_BF16, 2e-2)], ids=["f32", "bf16"])
@pytest.mark.parametrize("L,n", [((2, 2, 2, 2), 1), ((4, 4, 2, 2), 3), ((6, 10, 2, 14), 2), ((12, 10, 14, 16), 3)])
def test_mixing_tiles(L, n, arith, bar):
    U = S.gauge_links(L, 0.3, 81)
    ctx = P.Context(L, 0.124, 0.01)
    ctx.set_gauge(torch.from_numpy(U).to("cuda:0"))
    rng = np.random.default_rng(82)
    W1, W2 = (0.3 * (rng.standard_normal((9, 10, 4, 4)) + 1j * rng.standard_normal((9, 10, 4, 4))) for _ in range(2))
    ctx.ptc_set_arith(arith)
    ctx.ptc_set_weights(W1, W2)
    psi = S.random_spinor(L, 83, n)
    dpsi = torch.from_numpy(psi).to("cuda:0")
    out = torch.zeros_like(dpsi)
    ctx.ptc_apply(out, dpsi, n)
    for r in range(n):
        one = torch.zeros_like(dpsi[r:r + 1])
        ctx.ptc_apply(one, dpsi[r:r + 1].contiguous(), 1)
        torch.cuda.synchronize()
        assert torch.equal(out[r:r + 1], one)
        ref = O.ptc_forward(L, -1, U, W1, W2, psi[r])
        assert np.abs(out[r].cpu().numpy() - ref).max() <= bar * np.abs(ref).max()
    ctx.close()
