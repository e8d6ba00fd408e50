"""The hopping kernel's block decomposition: 64 half-sites per block, the
right-hand sides of a block one after the other.

Checked where it can go wrong: half-lattices smaller than a block, with a
ragged last block and of whole blocks; extents whose division has no power of
two; one right-hand side per block (its own instantiation), several, all, and
groups that do not divide their number.  Every split gives the same bits (each
output is one fixed-order sum), and the FP64 result agrees with the oracle
within 1e-13 (the bar of the FP64 operators).
"""
import os

import numpy as np
import pytest

import oracle as O
import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402

DEV = "cuda:0"
DTYPE = {P.TM_F64: torch.float64, P.TM_F32: torch.float32, P.TM_F16: torch.float16, P.TM_BF16: torch.bfloat16}
# V/2 = 8 (under a block), 420 (ragged, 6 blocks and 36 sites), 1024 (whole)
LATS = [(2, 2, 2, 2), (6, 10, 2, 14), (4, 8, 4, 16)]


@pytest.mark.parametrize("params", [18, 12, 8])
@pytest.mark.parametrize("prec", [P.TM_F64, P.TM_F32, P.TM_F16, P.TM_BF16])
@pytest.mark.parametrize("L", LATS)
def test_every_split_of_the_right_hand_sides(L, prec, params, monkeypatch):
    n, kappa, eps = 7, 0.124, 0.0123
    U = S.gauge_links(L, 0.3, 17)
    ctx = P.Context(L, kappa, eps)
    ctx.set_gauge(torch.from_numpy(U).to(DEV))
    ctx.set_link_format(params)
    full = S.random_spinor(L, 23, n)
    dfull = torch.from_numpy(full).to(DEV)
    e, o = (torch.zeros(ctx.half_numel(prec, n), dtype=torch.uint8, device=DEV) for _ in range(2))
    ctx.pack(e, o, dfull, n, prec)
    for kind in (P.TM_RINV_HOP_OE, P.TM_SCHUR, P.TM_SCHUR_DAG):
        got = []
        for split in ("1", "2", "3", "7", None):
            if split is None:
                monkeypatch.delenv("TM_DSLASH_RHS_TILE", raising=False)
            else:
                monkeypatch.setenv("TM_DSLASH_RHS_TILE", split)
            out = torch.zeros_like(e)
            ctx.dslash(out, e, n, kind, 1, prec)
            torch.cuda.synchronize()
            got.append(out.view(DTYPE[prec]).view(n, 12, ctx.hs, 2)[:, :, :ctx.vh].cpu())
        for g in got[1:]:
            assert torch.equal(g, got[0]), (L, prec, params, kind)
        if prec == P.TM_F64 and kind == P.TM_SCHUR:
            par, V = O.site_parity(L), int(np.prod(L))
            sites = np.arange(V)[par == 0]
            for r in range(n):
                v = full[r].copy()
                v[par == 1] = 0
                ref = O.schur(L, kappa, eps, -1, U, v).reshape(V, 12)[sites].T
                h = got[0][r].numpy()
                h = h[..., 0] + 1j * h[..., 1]
                assert np.abs(h - ref).max() <= 1e-13 * np.abs(ref).max()
