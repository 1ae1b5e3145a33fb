"""Products on the LDS ring whose rows are whole 8-byte pieces: the last tile ends with the matrix, and its values are those of the
same product on rows padded to whole 16-byte pieces."""
import pytest
import torch

from paper_2102_02344_amd import binding as hb

DEV = "cuda"


def _cs(B, C, L):
    return (C * L, B * C * L, L, 1)


# B, Nb, Ci, Co, L: the smallest last tile (4 columns), one column short of whole, both operands with such rows (Ci = 260, 516)
SHAPES = [(1, 96, 256, 256, 260), (2, 48, 256, 512, 508), (3, 33, 260, 256, 300), (1, 50, 516, 256, 1020), (1, 196, 264, 256, 256 + 252)]


@pytest.mark.gpu
@pytest.mark.parametrize("B,Nb,Ci,Co,L", SHAPES)
def test_rows_of_8_bytes(B, Nb, Ci, Co, L):
    g = torch.Generator(device=DEV).manual_seed(L)
    r = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
    x, w, dy, bias = r(Nb, B * Ci, L), r(B, Co, Ci), r(Nb, B * Co, L), r(B, Co)
    y, dx = torch.full((Nb, B * Co, L), float("nan"), dtype=torch.bfloat16, device=DEV), torch.full((Nb, B * Ci, L), float("nan"), dtype=torch.bfloat16, device=DEV)
    hb.conv1x1_fwd(B, Nb, Ci, Co, L, hb.BF16, x, _cs(B, Ci, L), w, bias, y, _cs(B, Co, L), hb.ACT_RELU)
    hb.conv1x1_bwd(B, Nb, Ci, Co, L, hb.BF16, None, None, w, dy, _cs(B, Co, L), dx, _cs(B, Ci, L), None, None, None)

    P = L + 4                                              # the same rows, padded
    pad = lambda t: torch.nn.functional.pad(t, (0, 4)).contiguous()
    y2, dx2 = torch.empty(Nb, B * Co, P, dtype=torch.bfloat16, device=DEV), torch.empty(Nb, B * Ci, P, dtype=torch.bfloat16, device=DEV)
    hb.conv1x1_fwd(B, Nb, Ci, Co, P, hb.BF16, pad(x), _cs(B, Ci, P), w, bias, y2, _cs(B, Co, P), hb.ACT_RELU)
    hb.conv1x1_bwd(B, Nb, Ci, Co, P, hb.BF16, None, None, w, pad(dy), _cs(B, Co, P), dx2, _cs(B, Ci, P), None, None, None)
    for a, b, what in ((y, y2, "forward"), (dx, dx2, "data gradient")):
        b = b[:, :, :L].contiguous()
        assert torch.isfinite(a.float()).all(), what
        # (two tiles more may decide for a kernel that adds the bias last: half an ulp of the stored value then)
        d = (a.float() - b.float()).abs()
        assert (d <= b.float().abs() * 2.0 ** -7).all(), (what, float(d.max()))
        assert float((d > 0).float().mean()) < 1e-2, what
    # and against the definition, on one sample: a rounding to bf16 of an fp32 sum of K products
    n = Nb - 1
    for b in range(B):
        ref = w[b].double() @ x[n].view(B, Ci, L)[b].double() + bias[b].double()[:, None]
        tol = 2.0 ** -8 * ref.abs() + Ci * 2.0 ** -24 * (w[b].double().abs() @ x[n].view(B, Ci, L)[b].double().abs())
        assert ((y[n].view(B, Co, L)[b].double() - ref.clamp_min(0)).abs() <= tol).all()
        ref = w[b].double().t() @ dy[n].view(B, Co, L)[b].double()
        tol = 2.0 ** -8 * ref.abs() + Co * 2.0 ** -24 * (w[b].double().abs().t() @ dy[n].view(B, Co, L)[b].double().abs())
        assert ((dx[n].view(B, Ci, L)[b].double() - ref).abs() <= tol).all()
