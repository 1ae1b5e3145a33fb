"""Training BatchNorm whose channels stay on chip between its passes, where the number of four-element pieces a thread holds
or the size staged for rows of other lengths changes kernel: one piece short of a full thread and one past it, channels that fit
in part or not at all, launches of more channels than compute units, short rows whose places outnumber their elements."""
import pytest
import torch

from util import DT, TOL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


# (Nb, L): pieces a thread has at 256 threads (channels below 32 KB) and at 1024
BF16 = [(1, 5), (2, 6), (3200, 5), (1630, 6), (1, 2052), (4, 1028), (3, 1363), (5, 2049), (7, 2338), (4, 4096), (4, 4100), (10, 4096), (10, 4099), (17, 2411), (20, 4096),
        (20, 4101), (40, 4096), (41, 4095), (10, 1021), (8, 2541), (16, 2549)]
F32 = [(1, 5), (1600, 5), (850, 9), (1, 1024), (1, 4100), (3, 1363), (5, 1639), (2, 4096), (5, 4096), (5, 4099), (9, 4096), (9, 4099), (10, 4097), (17, 4095),
       (17, 4097), (20, 4096), (20, 4098), (41, 4097)]


@pytest.mark.parametrize("dtype,B,C,Nb,L", [("bf16", 2, 3, *s) for s in BF16] + [("f32", 2, 3, *s) for s in F32]
                         + [("f32", 2, 140, 10, 4100), ("bf16", 3, 100, 11, 4093)])
def test_batchnorm_pieces(hb, dtype, B, C, Nb, L):
    """Against float64 on the stored inputs.  Outputs: the storage tolerance (fp32: 2e-5 .. 3e-5 for the three rounded factors);
    sums: against the magnitude of their terms."""
    print(f"held pieces {dtype} B={B} C={C} Nb={Nb} L={L}", flush=True)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(Nb * 10000 + L)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    x, dy = (r(Nb, B * C, L) * 1.7 + 0.6).to(td), r(Nb, B * C, L).to(td)
    g, bt = 1.0 + 0.4 * r(B * C), 0.3 * r(B * C)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    sm, si, dg, db, s3 = (torch.empty(B * C, device="cuda") for _ in range(5))
    st = (C * L, B * C * L, L, 1)
    hb.bn_fwd(B, Nb, C, L, DT[dtype], x, st, g, bt, 1e-5, 0.1, None, None, sm, si, y, st, hb.ACT_LEAKY, 0.2)
    x64, ch = x.double(), lambda v: v.double()[None, :, None]
    mean, var = x64.mean((0, 2)), x64.var((0, 2), unbiased=False)
    inv = (var + 1e-5).rsqrt()
    xh = (x64 - ch(mean)) * ch(inv)
    pre = ch(g) * xh + ch(bt)
    rel = lambda a, b: ((a.double() - b).abs().max() / b.abs().max()).item()
    tol = TOL[dtype]
    assert rel(sm, mean) <= 1e-5 and rel(si, inv) <= 1e-5
    assert rel(y, torch.where(pre > 0, pre, 0.2 * pre)) <= max(tol, 2e-5)
    dy[pre.abs() <= 1e-5] = 0                              # within fp32 rounding of the kink either branch is right
    gr = dy.double() * torch.where(pre > 0, 1.0, 0.2)
    hb.bn_bwd(B, Nb, C, L, DT[dtype], x, st, dy, st, g, bt, sm, si, dx, st, dg, db, hb.ACT_LEAKY, 0.2, s3)
    s1, s2, m = gr.sum((0, 2)), (gr * xh).sum((0, 2)), Nb * L
    mag = gr.abs().sum((0, 2)).max()
    assert (db - s1).abs().max() <= 2e-5 * mag and (dg - s2).abs().max() <= 1e-4 * mag
    assert rel(dx, ch(g) * ch(inv) * (gr - ch(s1) / m - xh * ch(s2) / m)) <= max(tol, 3e-5)
    assert (s3 - dx.double().sum((0, 2))).abs().max() <= 1e-5 * dx.double().abs().sum((0, 2)).max()
    # in place, the same bits
    y2, dx2 = x.clone(), dy.clone()
    hb.bn_fwd(B, Nb, C, L, DT[dtype], y2, st, g, bt, 1e-5, 0.1, None, None, sm, si, y2, st, hb.ACT_LEAKY, 0.2)
    hb.bn_bwd(B, Nb, C, L, DT[dtype], x, st, dx2, st, g, bt, sm, si, dx2, st, dg, db, hb.ACT_LEAKY, 0.2, s3)
    assert torch.equal(y, y2) and torch.equal(dx, dx2)
