"""bfloat16 spinors are stored rounded to nearest even, NaN stays NaN: the
conversion of canonical fields over all kinds of FP32 values (ties, the largest
ones, denormals, infinities, NaN), and the store of the hopping kernel, whose
values are those of the FP32 kernel on the same input (unit links are exact in
every link format)."""
import numpy as np
import pytest

import synth as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - collected on CPU hosts
    pytest.skip("no HIP device", allow_module_level=True)

import paper_1309_2256_amd as P  # noqa: E402

DEV = "cuda:0"


def nearest_even(f):
    """The bits of FP32 values rounded to bfloat16 (0x7fc0 for every NaN)."""
    u = f.view(np.uint32).astype(np.uint64)
    r = ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    return np.where(np.isnan(f), np.uint16(0x7fc0), r)


def stored(t):
    b = t.cpu().numpy().view(np.uint16)
    nan = ((b & 0x7f80) == 0x7f80) & ((b & 0x7f) != 0)
    return np.where(nan, np.uint16(0x7fc0), b)


def test_conversion_of_canonical_fields():
    L = (6, 10, 2, 14)
    ctx = P.Context(L, 0.124, 0.01)
    n = ctx.V * 24
    rng = np.random.default_rng(91)
    u = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    ties = slice(0, n // 4)  # exactly between two neighbours, and beside
    u[ties] = (u[ties] & 0xffff0000) | rng.choice(np.array([0x7fff, 0x8000, 0x8001], np.uint32), n // 4)
    u[-8:] = [0x7f7fffff, 0x7f7f8000, 0x7f7f7fff, 0x7f800000, 0xff800000, 0x00000001, 0x00018000, 0x80000000]
    f = u.view(np.float32)
    with np.errstate(invalid="ignore"):  # signalling NaN among the random bits
        full = torch.from_numpy(f.astype(np.float64)).to(DEV)
    e, o = (torch.zeros(ctx.half_numel(P.TM_BF16), dtype=torch.uint8, device=DEV) for _ in range(2))
    ctx.pack(e, o, full, 1, P.TM_BF16)
    e32, o32 = (torch.zeros(ctx.half_numel(P.TM_F32), dtype=torch.uint8, device=DEV) for _ in range(2))
    ctx.pack(e32, o32, full, 1, P.TM_F32)
    torch.cuda.synchronize()
    for h, h32 in ((e, e32), (o, o32)):
        assert np.array_equal(stored(h), nearest_even(h32.cpu().numpy().view(np.float32)))
    ctx.close()


@pytest.mark.parametrize("params", [18, 12])
def test_store_of_the_hopping_kernel(params):
    L, n = (6, 10, 2, 14), 3
    ctx = P.Context(L, 0.1237, 0.0123)
    U = np.zeros((4, ctx.V, 3, 3), complex)
    U[:] = np.eye(3)
    ctx.set_gauge(torch.from_numpy(U).to(DEV))
    ctx.set_link_format(params)
    v = torch.from_numpy(S.random_spinor(L, 92, n)).to(DEV).reshape(-1)
    v[5], v[777], v[2222] = float("nan"), float("inf"), 3e38
    a, b = (torch.zeros(ctx.half_numel(P.TM_BF16, n), dtype=torch.uint8, device=DEV) for _ in range(2))
    ctx.pack(a, b, v, n, P.TM_BF16)
    for half in (a, b):
        x16 = half.view(torch.bfloat16)
        x32 = x16.float()
        o16, o32 = torch.zeros_like(x16), torch.zeros_like(x32)
        ctx.dslash(o16, x16, n, P.TM_RINV_HOP_OE, 1, P.TM_BF16)
        ctx.dslash(o32, x32, n, P.TM_RINV_HOP_OE, 1, P.TM_F32)
        torch.cuda.synchronize()
        assert np.array_equal(stored(o16.view(torch.uint16)), nearest_even(o32.cpu().numpy()))
    ctx.close()
