"""hfta_conv1x1_bn_pool_fwd against the operators it stands for: with the activated tensor stored, bit for bit
hfta_conv1x1_bn_fwd and hfta_maxpool_points; without, in fp32, hfta_conv1x1_fwd and hfta_bn_fwd_maxpool.

There the statistics come from per-tile sums (combined in float64) instead of shifted sums over the channel: the reference
is the float64 mean and variance of the z the call stored, at the rounding of one fp32 value plus that of the sum of a tile's
squares, 2^-20.  The pooled value is that of the oracle's formula on the call's own statistics: four fp32 roundings of terms
no larger than |gamma xhat| + |beta|, and the index must hold it to the same."""
import numpy as np
import pytest
import torch

import hfta_inputs as hi
from util import DT, TDT, conv_strides, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


def setup(B, Nb, Ci, Co, L, dtype):
    x = hi.snap(np.maximum(hi.normal(441, (Nb, B * Ci, L)) + 0.3, 0.0), dtype)
    w = hi.normal(442, (B * Co, Ci), dtype, 1.0 / np.sqrt(Ci))
    bias = hi.normal(443, (B * Co,), dtype, 2.0)
    g = (hi.normal(444, (B * Co,)) * 0.3 + 1.0).astype(np.float32)
    g[::3] = -np.abs(g[::3])
    bt = (hi.normal(445, (B * Co,)) * 0.3).astype(np.float32)
    bt[1::7] = -6.0                                          # clipped everywhere
    g[5 % len(g)] = 0.0
    return [dev(a, dtype) for a in (x, w, bias)] + [dev(a) for a in (g, bt)]


def outputs(B, Nb, Co, L, dtype, stored):
    nan = float("nan")
    o = dict(Z=torch.full((Nb, B * Co, L), nan, dtype=TDT[dtype], device="cuda"), V=torch.full((B, Nb, Co), nan, dtype=TDT[dtype], device="cuda"),
             idx=torch.full((B, Nb, Co), -1, dtype=torch.int32, device="cuda"),
             rm=torch.ones(B * Co, device="cuda"), rv=torch.ones(B * Co, device="cuda"),
             mean=torch.full((B * Co,), nan, device="cuda"), invstd=torch.full((B * Co,), nan, device="cuda"))
    if stored:
        o["Y"] = torch.full_like(o["Z"], nan)
    return o


def call(hb, dims, dtype, ins, o, act, slope, ws):
    B, Nb, Ci, Co, L = dims
    X, W, Bi, G, Bt = ins
    ys = conv_strides(B, Co, L)
    hb.conv1x1_bn_pool_fwd(B, Nb, Ci, Co, L, DT[dtype], X, conv_strides(B, Ci, L), W, Bi, G, Bt, 1e-5, 0.1, o["rm"], o["rv"], o["mean"],
                           o["invstd"], o["Z"], ys, o.get("Y"), ys if "Y" in o else None, o["V"], o["idx"], (Nb * Co, Co, 1), act, slope, ws)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("dims", [(2, 3, 64, 130, 1300), (1, 2, 136, 520, 260), (2, 2, 16, 24, 131), (1, 1, 8, 9, 3), (2, 8, 64, 130, 510), (1, 16, 72, 256, 333)])
def test_stored(hb, dtype, dims):
    B, Nb, Ci, Co, L = dims
    ins = setup(*dims, dtype)
    X, W, Bi, G, Bt = ins
    n = max(4, hb.conv1x1_bn_pool_fwd_workspace_bytes(*dims, DT[dtype]))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    a, b = outputs(B, Nb, Co, L, dtype, True), outputs(B, Nb, Co, L, dtype, True)
    call(hb, dims, dtype, ins, a, hb.ACT_RELU, 0.0, ws)
    ys = conv_strides(B, Co, L)
    hb.conv1x1_bn_fwd(B, Nb, Ci, Co, L, DT[dtype], X, conv_strides(B, Ci, L), W, Bi, G, Bt, 1e-5, 0.1, b["rm"], b["rv"], b["mean"],
                      b["invstd"], b["Z"], ys, b["Y"], ys, hb.ACT_RELU, 0.0, ws)
    hb.maxpool_points(B, Nb, Co, L, DT[dtype], b["Y"], ys, b["V"], b["idx"], (Nb * Co, Co, 1))
    for k in a:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("with_ws", [True, False])
@pytest.mark.parametrize("act,slope", [(0, 0.0), (1, 0.0), (2, 0.2), (2, 0.0), (2, -0.5)])
@pytest.mark.parametrize("dims", [(4, 16, 70, 260, 1030), (2, 3, 64, 130, 300), (1, 2, 8, 65, 65), (1, 1, 5, 3, 4), (2, 2, 3, 70, 130)])
def test_pooled_only_f32(hb, dims, act, slope, with_ws):
    B, Nb, Ci, Co, L = dims
    ins = setup(*dims, "f32")
    ws = torch.empty(hb.conv1x1_bn_pool_fwd_workspace_bytes(*dims, 0), dtype=torch.uint8, device="cuda") if with_ws else None
    o = outputs(B, Nb, Co, L, "f32", False)
    call(hb, dims, "f32", ins, o, act, slope, ws)
    ref = torch.full_like(o["Z"], float("nan"))
    hb.conv1x1_fwd(B, Nb, Ci, Co, L, 0, ins[0], conv_strides(B, Ci, L), ins[1], ins[2], ref, conv_strides(B, Co, L))
    z = host(o["Z"]).astype(np.float64)
    assert np.abs(z - host(ref)).max() <= 2.0 ** -18 * np.abs(z).max()        # another tile may take the product
    g, bt = host(ins[3]).astype(np.float64), host(ins[4]).astype(np.float64)
    mean, var = z.mean(axis=(0, 2)), z.var(axis=(0, 2))
    # without a workspace, and under four input channels (single-element loads, an epilogue without sums): shifted sums in
    # fp32, hfta_bn_fwd_maxpool's own, at that operator's tolerance
    tol = 2.0 ** -20 if with_ws and Ci >= 4 else 1e-5
    gm, gi = host(o["mean"]).astype(np.float64), host(o["invstd"]).astype(np.float64)
    assert np.all(np.abs(gm - mean) <= tol * (np.abs(mean) + np.sqrt(var)))
    inv = 1.0 / np.sqrt(var + 1e-5)
    assert np.all(np.abs(gi - inv) <= tol * inv)
    m = Nb * L
    assert np.allclose(host(o["rm"]), 0.9 + 0.1 * mean, rtol=0, atol=1e-5 * (1 + np.abs(mean).max()))
    assert np.allclose(host(o["rv"]), 0.9 + 0.1 * var * m / max(m - 1, 1), rtol=1e-5, atol=1e-6)
    pre = g[:, None] * (z - gm[:, None]) * gi[:, None] + bt[:, None]
    y = pre if act == 0 else np.where(pre > 0, pre, (slope if act == 2 else 0.0) * pre)
    t3 = lambda a: a.reshape(Nb, B, Co).transpose(1, 0, 2)
    lim = 4 * 2.0 ** -24 * (np.abs(pre).max(axis=2) + np.abs(bt) + np.abs(g * gi) * np.abs(z).max(axis=2))
    idx = host(o["idx"]).transpose(1, 0, 2).reshape(Nb, B * Co, 1)
    assert idx.min() >= 0 and idx.max() < L
    assert np.all(np.abs(host(o["V"]) - t3(y.max(axis=2))) <= t3(lim))
    assert np.all(np.take_along_axis(y, idx.astype(np.int64), axis=2)[:, :, 0] >= y.max(axis=2) - lim)
    flat = (y.max(axis=2) == y.min(axis=2))
    assert np.all(idx[:, :, 0][flat] == 0)


@pytest.mark.parametrize("act,slope", [(0, 0.0), (1, 0.0), (2, 0.2)])
@pytest.mark.parametrize("dims", [(4, 16, 72, 260, 1028), (4, 16, 70, 260, 1030), (1, 2, 8, 65, 65)])
def test_channels_that_are_not_numbers_f32(hb, dims, act, slope):
    """NaN and infinities in z (from weights, so in some channels only; from one point, so in all of a model): values and
    indices of those channels are the two operators' own, the others stay finite."""
    B, Nb, Ci, Co, L = dims
    ins = setup(*dims, "f32")
    nan, inf = float("nan"), float("inf")
    ins[1][3, 1], ins[1][10, 2], ins[1][11, 2] = nan, inf, -inf
    if B > 1:
        ins[0][Nb // 2, Ci + 5, L - 1] = nan
        ins[0][1, 2 * Ci + 6, 7] = inf
    ws = torch.empty(hb.conv1x1_bn_pool_fwd_workspace_bytes(*dims, 0), dtype=torch.uint8, device="cuda")
    a, b = outputs(B, Nb, Co, L, "f32", False), outputs(B, Nb, Co, L, "f32", False)
    call(hb, dims, "f32", ins, a, act, slope, ws)
    X, W, Bi, G, Bt = ins
    ys = conv_strides(B, Co, L)
    hb.conv1x1_fwd(B, Nb, Ci, Co, L, 0, X, conv_strides(B, Ci, L), W, Bi, b["Z"], ys)
    hb.bn_fwd_maxpool(B, Nb, Co, L, 0, b["Z"], ys, G, Bt, 1e-5, 0.1, b["rm"], b["rv"], b["mean"], b["invstd"], b["V"], b["idx"],
                      (Nb * Co, Co, 1), act, slope)
    bad = ~torch.isfinite(b["mean"])
    assert bad.any() and not bad.all() and torch.equal(bad, ~torch.isfinite(a["mean"]))
    bad = bad.view(B, 1, Co).expand(B, Nb, Co)
    assert torch.equal(a["idx"][bad], b["idx"][bad])
    assert torch.equal(torch.nan_to_num(a["V"][bad], 7.0), torch.nan_to_num(b["V"][bad], 7.0))
    assert torch.isfinite(a["V"][~bad]).all()
