"""Fused Linear at the sizes the GEMM kernel with loads straight into LDS takes (few output tiles under a
reduction of at least five 64-element k-tiles): each of its three tiles, edges and remainders of a tile in
every dimension, the fewest and the most k-tiles, and the sizes one step outside.

Reference: float64 products of the same bf16 values.  Bound per element: the fp32 accumulation of K exact
products, at most K 2^-23 sum|a||b| in any order, and for bf16 outputs one rounding, 2^-8 of the value."""
import numpy as np
import pytest
import torch

import hfta_inputs as hi
from util import dev, host

pytestmark = pytest.mark.gpu
U = 2.0 ** -23


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


def within(got, ref, mag, K, bf16, what):
    d = np.abs(host(got).reshape(ref.shape) - ref)
    lim = K * U * mag + (2.0 ** -8 * np.abs(ref) if bf16 else 0.0) + 1e-30
    assert np.all(np.isfinite(d)), what
    assert (d <= lim).all(), (what, float((d / lim).max()))


@pytest.mark.parametrize("B,M,Fx,Fy", [
    (2, 33, 320, 64),        # 64 x 64 tiles, five k-tiles forward, rows past a half tile
    (1, 1, 264, 8),          # one row, one column piece, a last k-tile of one piece
    (2, 200, 328, 520),      # remainders in every dimension
    (3, 64, 8192, 72),       # the longest reduction (128 k-tiles)
    (3, 64, 8200, 72),       # one past it: the split path
    (5, 693, 384, 1000),     # 128 x 64 tiles backward
    (4, 1500, 392, 520),     # 128 x 128 tiles
    (1, 321, 1024, 1024),
    (2, 96, 327, 65),        # not whole pieces: the other kernels
])
def test_linear_forward_backward(hb, B, M, Fx, Fy):
    x = hi.normal(501, (B, M, Fx), "bf16")
    w = hi.snap(hi.normal(502, (B, Fx, Fy)) * 0.1, "bf16")
    bias = hi.normal(503, (B, Fy), "bf16")
    dy = hi.normal(504, (B, M, Fy), "bf16")
    X, W, Bi, dY = (dev(a, "bf16") for a in (x, w, bias, dy))
    x64, w64, b64, dy64 = (np.asarray(a, np.float64) for a in (x, w, bias, dy))
    aw, ax, ad = np.abs(w64), np.abs(x64), np.abs(dy64)
    lin = x64 @ w64 + b64[:, None, :]
    mag = ax @ aw + np.abs(b64)[:, None, :]
    ws = torch.empty(max(4, hb.linear_fwd_workspace_bytes(B, M, Fx, Fy, 1), hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, 1)),
                     dtype=torch.uint8, device="cuda")
    nan = float("nan")
    for act, ref in ((hb.ACT_NONE, lin), (hb.ACT_LEAKY, np.where(lin > 0, lin, 0.2 * lin))):
        Y, Y2 = (torch.full((B, M, Fy), nan, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        hb.linear_fwd(B, M, Fx, Fy, 1, X, W, Bi, Y, act, 0.2)
        within(Y, ref, mag, Fx + 1, True, f"forward act {act}")
        hb.linear_fwd_ws(B, M, Fx, Fy, 1, X, W, Bi, Y2, act, 0.2, ws)
        within(Y2, ref, mag, Fx + 1, True, f"forward with workspace act {act}")
    dX = torch.full((B, M, Fx), nan, dtype=torch.bfloat16, device="cuda")
    dW = torch.full((B, Fx, Fy), nan, device="cuda")
    db = torch.full((B, Fy), nan, device="cuda")
    hb.linear_bwd(B, M, Fx, Fy, 1, X, W, dY, dX, dW, db, ws)
    within(dX, dy64 @ w64.transpose(0, 2, 1), ad @ aw.transpose(0, 2, 1), Fy, True, "data gradient")
    within(dW, x64.transpose(0, 2, 1) @ dy64, ax.transpose(0, 2, 1) @ ad, M, False, "weight gradient")
    within(db, dy64.sum(1), ad.sum(1), M, False, "bias gradient")


@pytest.mark.parametrize("B,M,Fx,Fy", [(5, 693, 384, 1536), (1, 4096, 512, 512)])
@pytest.mark.parametrize("off", [0, 4, 1])
def test_weight_gradient_by_alignment(hb, B, M, Fx, Fy, off):
    """Operands that start on 16 bytes take the kernel unsplit and need no workspace; the same shape 8 or 2 bytes further
    on, which it does not take, is split over the workspace that the query asks for."""
    def place(seed, shape):
        n = int(np.prod(shape))
        return hi.normal(seed, shape, "bf16"), torch.empty(n + 8, dtype=torch.bfloat16, device="cuda")[off:off + n].view(shape)
    (x, X), (dy, dY) = place(511, (B, M, Fx)), place(512, (B, M, Fy))
    X.copy_(dev(x, "bf16"))
    dY.copy_(dev(dy, "bf16"))
    ws = torch.full((hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, 1),), 0xff, dtype=torch.uint8, device="cuda")
    assert ws.numel() >= 2 * B * Fx * Fy * 4
    dW, db = torch.full((B, Fx, Fy), float("nan"), device="cuda"), torch.full((B, Fy), float("nan"), device="cuda")
    hb.linear_bwd(B, M, Fx, Fy, 1, X, None, dY, None, dW, db, None if off == 0 else ws)
    x64, dy64 = np.asarray(x, np.float64), np.asarray(dy, np.float64)
    within(dW, x64.transpose(0, 2, 1) @ dy64, np.abs(x64).transpose(0, 2, 1) @ np.abs(dy64), M, False, "weight gradient")
    within(db, dy64.sum(1), np.abs(dy64).sum(1), M, False, "bias gradient")
    assert bool((ws != 0xff).any()) == (off != 0)
    if off:
        with pytest.raises(hb.HftaError):
            hb.linear_bwd(B, M, Fx, Fy, 1, X, None, dY, None, dW, db, None)


@pytest.mark.parametrize("M,Fx,Fy,models", [
    (300, 64, 72, (1, 3)),           # 64 x 64 tiles
    (693, 384, 1000, (1, 5)),        # 64 x 64 for one model, 128 x 64 for five
    (1501, 392, 520, (1, 4)),        # 64 x 64 and 128 x 128
    (600, 512, 2048, (1, 2, 12)),    # ... and the 256 x 256 kernel
    (2048, 256, 8192, (2, 8)),
])
def test_bias_gradient_is_one_sum(hb, M, Fx, Fy, models):
    """A model's bias gradient has the same bits however many models it is trained with and whether or not the weight
    gradient is asked for: rows r, r + 64, r + 128, .. are added in order, then the 64 sums in order."""
    B = max(models)
    x, dy = dev(hi.normal(521, (B, M, Fx), "bf16"), "bf16"), dev(hi.normal(522, (B, M, Fy), "bf16"), "bf16")
    chains = torch.zeros(B, 64, Fy)
    rows = dy.float().cpu()
    for r in range(M):
        chains[:, r % 64] += rows[:, r]
    ref = torch.zeros(B, Fy)
    for k in range(64):
        ref += chains[:, k]
    for n in models:
        ws = torch.empty(max(4, hb.linear_bwd_workspace_bytes(n, M, Fx, Fy, 1)), dtype=torch.uint8, device="cuda")
        for dW in (None, torch.empty(n, Fx, Fy, device="cuda")):
            db = torch.full((n, Fy), float("nan"), device="cuda")
            hb.linear_bwd(n, M, Fx, Fy, 1, None if dW is None else x, None, dy, None, dW, db, ws)
            assert torch.equal(db.cpu(), ref[:n]), (n, dW is None)
