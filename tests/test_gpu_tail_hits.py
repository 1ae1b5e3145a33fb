"""Backward of the one-operator tail where the argmax points crowd: more hits in a 128-point tile than are staged at a
time, all on one point, on the edges of tiles and of 32-column blocks, none at all in a tile; 1 to 1024 channels, both tile
depths, more samples than the coefficient kernel's eight rows of eight.

The indices are given (they need not be the maximum's), z at them is the float64 product, so the reference is the oracle's
composition on the same indices; tolerances are the operator's own test's."""
import numpy as np
import pytest
import torch

import hfta_inputs as hi
from oracle import array as oa
from util import DT, TOL, check, conv_strides, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


def indices(kind, r, shape, L):
    if kind == "one point":
        return np.full(shape, min(L - 1, 77))
    if kind == "one tile":
        return r.integers(128, min(L, 256), shape)
    if kind == "edges":
        return r.choice([i for i in (0, 31, 32, 63, 64, 127, 128, 255, L - 1) if i < L], shape)
    return np.minimum(r.integers(0, (L + 127) // 128, shape) // 2 * 256 + 5, L - 1)      # every other tile: one column


@pytest.mark.parametrize("kind", ["one point", "one tile", "edges", "every other"])
@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(1, 2, 128, 1024, 300), (2, 3, 64, 129, 257), (1, 70, 8, 17, 132), (1, 1, 72, 1, 516)])
def test_crowded_hits(hb, B, Nb, Ci, Co, L, kind):
    r = np.random.default_rng(Co)
    x = hi.snap(np.maximum(hi.normal(341, (Nb, B * Ci, L)) + 0.3, 0.0), "bf16")
    w = hi.normal(342, (B * Co, Ci), "bf16", 1.0 / np.sqrt(Ci))
    bias = hi.normal(343, (B * Co,), "bf16", 0.1)
    g = (hi.normal(344, (B * Co,)) * 0.3 + 1.0).astype(np.float32)
    bt = (hi.normal(345, (B * Co,)) * 0.3).astype(np.float32)
    dv = hi.normal(346, (B, Nb, Co), "bf16")
    idx = indices(kind, r, (Nb, B * Co), L).astype(np.int32)
    z = oa.conv1x1_fwd(B, x, w, bias)
    zh = np.take_along_axis(z, idx[:, :, None].astype(np.int64), axis=2)[:, :, 0]
    t3 = lambda a: np.ascontiguousarray(a.reshape(Nb, B, Co).transpose(1, 0, 2))
    mean = z.mean(axis=(0, 2)).astype(np.float32)
    invstd = (1.0 / np.sqrt(z.var(axis=(0, 2)) + 1e-5)).astype(np.float32)
    ref = oa.conv1x1_bn_maxpool_bwd(B, x, w, bias, g, bt, mean, invstd, dv.transpose(1, 0, 2).reshape(Nb, B * Co), idx, 0, 0.0)
    X, W, Bi, dV, I, ZH = dev(x, "bf16"), dev(w, "bf16"), dev(bias, "bf16"), dev(dv, "bf16"), dev(t3(idx)), dev(t3(zh).astype(np.float32))
    G, Bt, SM, SI = dev(g), dev(bt), dev(mean), dev(invstd)
    dX = torch.full(x.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    dW, dB0, dG, dBt = (torch.full((n,), float("nan"), device="cuda") for n in (B * Co * Ci, B * Co, B * Co, B * Co))
    ws = torch.empty(hb.conv1x1_bn_maxpool_workspace_bytes(B, Nb, Ci, Co, L, DT["bf16"]), dtype=torch.uint8, device="cuda")
    sx = conv_strides(B, Ci, L)
    hb.conv1x1_bn_maxpool_bwd(B, Nb, Ci, Co, L, DT["bf16"], X, sx, W, Bi, None, None, ZH, None, dV, I.int(), (Nb * Co, Co, 1), G, Bt,
                              SM, SI, dX, sx, dW, dB0, dG, dBt, 0, 0.0, ws)
    sc = np.abs(dv).sum(axis=1).max()
    assert np.abs(host(dG) - ref[3]).max() <= 2e-4 * max(np.abs(ref[3]).max(), sc * 1e-2)
    assert np.abs(host(dBt) - ref[4]).max() <= 2e-4 * max(np.abs(ref[4]).max(), sc * 1e-2)
    check(host(dX), ref[0], TOL["bf16"], "dX")
    check(host(dW).reshape(ref[1].shape), ref[1], 2e-4, "dW")


@pytest.mark.parametrize("act", [0, 1, 2])
def test_zero_scale_pools_the_shift(hb, act):
    """gamma == 0: every point's activated value is act(beta), the first point's index; a positive beta is not clipped."""
    B, Nb, Ci, Co, L = 1, 2, 16, 24, 300
    X = dev(hi.snap(np.abs(hi.normal(351, (Nb, Ci, L))), "bf16"), "bf16")
    W, bt = dev(hi.normal(352, (Co, Ci), "bf16"), "bf16"), hi.normal(353, (Co,)).astype(np.float32)
    G, Bt = torch.zeros(Co, device="cuda"), dev(bt)
    SM, SI, ZH = (torch.empty(n, device="cuda") for n in (Co, Co, Nb * Co))
    V = torch.full((B, Nb, Co), float("nan"), dtype=torch.bfloat16, device="cuda")
    I = torch.full((B, Nb, Co), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(hb.conv1x1_bn_maxpool_workspace_bytes(B, Nb, Ci, Co, L, DT["bf16"]), dtype=torch.uint8, device="cuda")
    hb.conv1x1_bn_maxpool_fwd(B, Nb, Ci, Co, L, DT["bf16"], X, conv_strides(B, Ci, L), W, None, G, Bt, 1e-5, 0.1, None, None, SM, SI, V, I,
                              (Nb * Co, Co, 1), ZH, None, act, 0.2, ws)
    ref = bt if act == 0 else np.where(bt > 0, bt, (0.2 if act == 2 else 0.0) * bt)
    assert (bt > 0).any() and int(I.abs().max()) == 0
    assert torch.equal(V[0].cpu(), torch.from_numpy(ref.astype(np.float32)).bfloat16().expand(Nb, Co))


@pytest.mark.parametrize("near", ["rounding of the value", "rounding of point 0"])
@pytest.mark.parametrize("L", [516, 257])
def test_mask_is_the_pooled_values(hb, L, near):
    """Shifts that bring a sample's maximum within rounding of zero: gradient passes where, and only where, a positive value was
    pooled, so with a gradient of one dbeta counts them.  "Point 0": its z is 2^-16 below the maximum's, and recomputed one
    product after the other through partial sums of about 64 it comes out above in some channels."""
    B, Nb, Ci, Co = 2, 3, 64, 512
    x = hi.normal(361, (Nb, B, Ci, L))
    if near == "rounding of point 0":
        x[..., 1] *= 8.0
        x[..., 2:] *= 0.0625
        x[:, :, 1, 1], x[:, :, Ci - 1, 1] = 512.0, -512.0
        x[:, :, 0, 1] = 2.0 ** -6
        x[..., 0] = x[..., 1]
        x[:, :, 0, 0] = 0.0
    x = hi.snap(x.reshape(Nb, B * Ci, L).astype(np.float32), "bf16")
    w = hi.normal(362, (B * Co, Ci), "bf16", 1.0 / np.sqrt(Ci))
    if near == "rounding of point 0":
        w[:, 0] = 2.0 ** -10
        w[:, Ci - 1] = w[:, 1]
    g = np.abs(hi.normal(363, (B * Co,)) * 0.3 + 1.0).astype(np.float32) + np.float32(0.1)
    X, W, G = dev(x, "bf16"), dev(w, "bf16"), dev(g)
    SM, SI = torch.empty(B * Co, device="cuda"), torch.empty(B * Co, device="cuda")
    V, I = torch.empty(B, Nb, Co, dtype=torch.bfloat16, device="cuda"), torch.empty(B, Nb, Co, dtype=torch.int32, device="cuda")
    Z, M = torch.empty(B, Nb, Co, device="cuda"), torch.empty(hb.conv1x1_bn_maxpool_saved_floats(B, Ci, Co), device="cuda")
    ws = torch.empty(hb.conv1x1_bn_maxpool_workspace_bytes(B, Nb, Ci, Co, L, DT["bf16"]), dtype=torch.uint8, device="cuda")
    sx, vs = conv_strides(B, Ci, L), (Nb * Co, Co, 1)

    def forward(beta, act):
        hb.conv1x1_bn_maxpool_fwd(B, Nb, Ci, Co, L, DT["bf16"], X, sx, W, None, G, beta, 1e-5, 0.1, None, None, SM, SI, V, I, vs, Z, M,
                                  act, 0.0, ws)

    forward(torch.zeros(B * Co, device="cuda"), hb.ACT_NONE)
    z, mean, invstd = Z[:, 0].reshape(-1).clone(), SM.clone(), SI.clone()
    if L % 4:
        z = z.bfloat16().float()
    beta = -((G * invstd) * (z - mean))
    ulps = torch.tensor([-1, 0, 0, 1], device="cuda", dtype=torch.int32).repeat(B * Co // 4)
    beta = (beta.view(torch.int32) + ulps).view(torch.float32)
    forward(beta, hb.ACT_RELU)
    dX, dV = torch.empty_like(X), torch.ones_like(V)
    dW, dG, dBt = (torch.empty(n, device="cuda") for n in (B * Co * Ci, B * Co, B * Co))
    hb.conv1x1_bn_maxpool_bwd(B, Nb, Ci, Co, L, DT["bf16"], X, sx, W, None, None, None, Z, M, dV, I, vs, G, beta, SM, SI, dX, sx, dW,
                              None, dG, dBt, hb.ACT_RELU, 0.0, ws)
    assert torch.equal(dBt.view(B, Co), (V.float() > 0).float().sum(1))
