"""The site contraction fused with the transform along x: whole x rows per
block.  Sizes where the row grouping can go wrong: rows that divide a block
(2, 16), that leave idle threads (6, 34), of exactly a block (256) and longer
than one (258, the unfused path), and row counts that fill no group; against
the oracle's site-by-site densities and Fourier sums within 1e-13, the bar of
the FP64 contractions."""
import numpy as np
import pytest

import oracle as O
import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402

EST = P.TM_EST_STD | P.TM_EST_ONE_END
ORDER = (O.EST_STD, O.EST_ONE_END)


@pytest.mark.parametrize("L,p2max", [((2, 4, 6, 2), 0), ((16, 6, 4, 2), 2), ((6, 10, 4, 6), 3),
                                     ((34, 4, 4, 2), 1), ((256, 4, 2, 2), 0), ((258, 4, 2, 2), 0)])
def test_rows_match_oracle(L, p2max):
    kappa, eps, nrhs = 0.124, 0.0123, 2
    U = S.gauge_links(L, 0.3, 41)
    ctx = P.Context(L, kappa, eps)
    ctx.set_gauge(torch.from_numpy(U).to("cuda:0"))
    eta, s = S.random_spinor(L, 42, nrhs), S.random_spinor(L, 43, nrhs)
    moms = O.momenta(p2max)
    got = ctx.contract_momentum(*(torch.from_numpy(f).to("cuda:0") for f in (eta, s)), nrhs, EST, p2max, 1,
                                derivative=1)
    ref = [O.contract_insertions(L, kappa, eps, -1, U, eta[r], s[r], EST, True, moms) for r in range(nrhs)]
    for k, e in enumerate(ORDER):
        want = sum(x[e] for x in ref)
        assert np.abs(got[k] - want).max() <= 1e-13 * np.abs(want).max(), (L, e)
