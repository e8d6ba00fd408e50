"""One right-hand side per block: half-precision spinors with FP32 links take the
form of several there, the other precisions their own.  Every split gives the same
bits, on half-lattices below a block, ragged and of whole blocks."""
import pytest

import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402

DEV = "cuda:0"
DTYPE = {P.TM_F16: torch.float16, P.TM_BF16: torch.bfloat16}


@pytest.mark.parametrize("prec", [P.TM_F16, P.TM_BF16])
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (6, 10, 2, 14), (4, 8, 4, 16)])
def test_fp32_links_of_half_spinors(L, prec, monkeypatch):
    n = 5
    ctx = P.Context(L, 0.124, 0.0123)
    ctx.set_gauge(torch.from_numpy(S.gauge_links(L, 0.3, 17)).to(DEV))
    e, o = (torch.zeros(ctx.half_numel(prec, n), dtype=torch.uint8, device=DEV) for _ in range(2))
    ctx.pack(e, o, torch.from_numpy(S.random_spinor(L, 23, n)).to(DEV), n, prec)
    for kind in (P.TM_RINV_HOP_OE, P.TM_SCHUR, P.TM_SCHUR_DAG):
        got = []
        for split in ("1", "2", "3", "5"):
            monkeypatch.setenv("TM_DSLASH_RHS_TILE", split)
            out = torch.zeros_like(e)
            ctx.dslash(out, e, n, kind, 1, prec, P.TM_F32)
            torch.cuda.synchronize()
            got.append(out.view(DTYPE[prec]).view(n, 12, ctx.hs, 2)[:, :, :ctx.vh].cpu())
        for g in got[1:]:
            assert torch.equal(g, got[0]), (L, prec, kind)
    ctx.close()
