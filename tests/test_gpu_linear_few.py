"""Linear layers of few rows with the operators beside them: the bits of the single operators, at tile edges and remainders."""
import ctypes as C

import pytest
import torch

from paper_2102_02344_amd import binding as hb

DEV = "cuda"


def _rand(g, *shape, scale=1.0):
    return ((torch.rand(shape, generator=g) * 2 - 1) * scale).to(torch.bfloat16).to(DEV)


def _f32(g, *shape):
    return (torch.rand(shape, generator=g) + 0.5).to(DEV)


def _same(a, b, what):
    assert torch.equal(a.view(torch.int32) if a.dtype == torch.float32 else a.view(torch.int16),
                       b.view(torch.int32) if b.dtype == torch.float32 else b.view(torch.int16)), what


SHAPES = [(1, 1, 8, 8), (2, 2, 96, 16), (3, 13, 1024, 512), (16, 16, 1216, 40), (5, 17, 72, 264), (8, 32, 512, 256), (40, 31, 136, 72)]


@pytest.mark.gpu
@pytest.mark.parametrize("B,M,Fx,Fy", SHAPES)
@pytest.mark.parametrize("drop", [False, True])
def test_linear_batchnorm(B, M, Fx, Fy, drop):
    g = torch.Generator().manual_seed(B * 1000 + M)
    assert hb.linear_few_supported(B, M, Fx, Fy, hb.BF16)
    x, w, bias = _rand(g, B, M, Fx), _rand(g, B, Fx, Fy, scale=Fx ** -0.5), _rand(g, B, Fy)
    gamma, beta = _f32(g, B, Fy), _f32(g, B, Fy) - 1.0
    mask = (torch.rand((B, M, Fy), generator=g) < 0.7).to(torch.uint8).to(DEV) if drop else None
    ls = (M * Fy, Fy, 1, 1)

    def outputs():
        o = dict(z=torch.empty(B, M, Fy), y=torch.empty(B, M, Fy), yd=torch.empty(B, M, Fy))
        o = {k: v.to(torch.bfloat16).to(DEV) for k, v in o.items()}
        return o, dict(rm=torch.full((B, Fy), 0.25, device=DEV), rv=torch.full((B, Fy), 1.5, device=DEV),
                       mean=torch.empty(B, Fy, device=DEV), invstd=torch.empty(B, Fy, device=DEV))

    (o1, s1), (o2, s2) = outputs(), outputs()
    ws = torch.empty(max(4, hb.linear_fwd_workspace_bytes(B, M, Fx, Fy, hb.BF16)), dtype=torch.uint8, device=DEV)
    hb.linear_fwd_ws(B, M, Fx, Fy, hb.BF16, x, w, bias, o1["z"], workspace=ws)
    hb.bn_fwd(B, M, Fy, 1, hb.BF16, o1["z"], ls, gamma, beta, 1e-5, 0.1, s1["rm"], s1["rv"], s1["mean"], s1["invstd"], o1["y"], ls,
              hb.ACT_RELU)
    if drop:
        hb.dropout(B * M * Fy, hb.BF16, o1["y"], mask, 0.3, o1["yd"])
    hb.linear_bn_fwd(B, M, Fx, Fy, hb.BF16, x, w, bias, gamma, beta, 1e-5, 0.1, s2["rm"], s2["rv"], s2["mean"], s2["invstd"], o2["z"],
                     o2["y"], hb.ACT_RELU, 0.0, mask, 0.3 if drop else 0.0, o2["yd"] if drop else None)
    for k in ("z", "y") + (("yd",) if drop else ()):
        _same(o1[k], o2[k], k)
    for k in s1:
        _same(s1[k], s2[k], k)

    # backward: this Linear's gradients, and on through a BatchNorm below it (of Fx channels)
    dy, zb = _rand(g, B, M, Fy, scale=0.1), _rand(g, B, M, Fx)
    gb, bb = _f32(g, B, Fx), _f32(g, B, Fx) - 1.0
    mean, invstd = zb.float().mean(1).contiguous(), _f32(g, B, Fx)
    maskb = (torch.rand((B, M, Fx), generator=g) < 0.7).to(torch.uint8).to(DEV) if drop else None
    lx = (M * Fx, Fx, 1, 1)
    wb = torch.empty(max(4, hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.BF16)), dtype=torch.uint8, device=DEV)
    bf = dict(dtype=torch.bfloat16, device=DEV)
    dx, dd, dz = (torch.empty(B, M, Fx, **bf) for _ in range(3))
    dw, db = torch.empty(B, Fx, Fy, device=DEV), torch.empty(B, Fy, device=DEV)
    sums = [torch.empty(B, Fx, device=DEV) for _ in range(3)]
    hb.linear_bwd(B, M, Fx, Fy, hb.BF16, x, w, dy, dx, dw, db, wb)
    if drop:
        hb.dropout(B * M * Fx, hb.BF16, dx, maskb, 0.3, dd)
    hb.bn_bwd(B, M, Fx, 1, hb.BF16, zb, lx, dd if drop else dx, lx, gb, bb, mean, invstd, dz, lx, sums[0], sums[1], hb.ACT_RELU, 0.0, sums[2])
    dx2, dz2 = torch.empty(B, M, Fx, **bf), torch.empty(B, M, Fx, **bf)
    dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
    dw3 = torch.empty_like(dw)
    sums2 = [torch.empty(B, Fx, device=DEV) for _ in range(3)]
    hb.linear_bwd_bn(B, M, Fx, Fy, hb.BF16, x, w, dy, dx2, dw2, db2)
    hb.linear_bwd_bn(B, M, Fx, Fy, hb.BF16, x, w, dy, dz2, dw3, None, zb, gb, bb, mean, invstd, hb.ACT_RELU, 0.0, maskb,
                     0.3 if drop else 0.0, *sums2)
    for a, b, what in ((dx, dx2, "dX"), (dw, dw2, "dW"), (dw, dw3, "dW"), (db, db2, "dbias"), (dz, dz2, "dZ")):
        _same(a, b, what)
    for a, b, what in zip(sums, sums2, ("dgamma", "dbeta", "sum of dZ")):
        _same(a, b, what)


@pytest.mark.gpu
@pytest.mark.parametrize("B,M,Fx,K", [(1, 1, 8, 8), (3, 13, 256, 16), (8, 32, 256, 16), (2, 17, 1000, 32)])
def test_linear_cross_entropy(B, M, Fx, K):
    g = torch.Generator().manual_seed(M)
    x, w, bias = _rand(g, B, M, Fx), _rand(g, B, Fx, K, scale=3 * Fx ** -0.5), _rand(g, B, K)
    labels = torch.randint(K, (B, M), generator=g, dtype=torch.int32).to(DEV)
    bf = dict(dtype=torch.bfloat16, device=DEV)
    z1, z2, d1, d2 = (torch.empty(B, M, K, **bf) for _ in range(4))
    l1, l2 = torch.empty(B, device=DEV), torch.empty(B, device=DEV)
    ws = torch.empty(max(4, hb.linear_fwd_workspace_bytes(B, M, Fx, K, hb.BF16)), dtype=torch.uint8, device=DEV)
    hb.linear_fwd_ws(B, M, Fx, K, hb.BF16, x, w, bias, z1, workspace=ws)
    hb.softmax_xent(B, M, K, hb.BF16, z1, labels, l1, d1)
    hb.linear_xent(B, M, Fx, K, hb.BF16, x, w, bias, z2, labels, l2, d2)
    for a, b, what in ((z1, z2, "logits"), (l1, l2, "loss"), (d1, d2, "dlogits")):
        _same(a, b, what)


def test_what_is_declined():
    ok = lambda *a: hb.linear_few_supported(*a)
    assert ok(8, 32, 1024, 512, hb.BF16) and ok(1, 1, 8, 8, hb.BF16)
    assert not ok(8, 33, 1024, 512, hb.BF16) and not ok(8, 32, 1024, 512, hb.F32)
    assert not ok(8, 32, 1028, 512, hb.BF16) and not ok(8, 32, 256, 9, hb.BF16) and not ok(16, 32, 1224, 512, hb.BF16) and not ok(1, 32, 1216, 40, hb.BF16)
    raw, one, off = hb.raw(), C.c_void_p(256), C.c_void_p(264)

    def bn(X=one, W=one, M=32, act=1, mask=None, Yd=None, p=0.0, rv=one):
        return raw.hfta_linear_bn_fwd(8, M, 256, 64, 1, X, W, None, one, one, 1e-5, 0.1, one, rv, one, one, one, one, act, 0.0, mask, p,
                                      Yd, None)
    assert bn(X=None) == hb.EINVAL and bn(rv=None) == hb.EINVAL and bn(mask=one) == hb.EINVAL and bn(mask=one, Yd=one, p=1.0) == hb.EINVAL
    assert bn(X=off) == hb.EUNSUPPORTED and bn(W=off) == hb.EUNSUPPORTED and bn(M=33) == hb.EUNSUPPORTED
    assert bn(act=hb.ACT_TANH) == hb.EUNSUPPORTED
    assert raw.hfta_linear_xent(8, 32, 256, 40, 1, one, one, None, one, one, one, one, None) == hb.EUNSUPPORTED
    assert raw.hfta_linear_xent(8, 32, 256, 16, 1, one, one, None, one, None, one, one, None) == hb.EINVAL

    def bwd(dY=one, M=32, Z=None, mean=one, mask=None, dsum=None, Fy=64):
        return raw.hfta_linear_bwd_bn(8, M, 256, Fy, 1, one, one, dY, one, one, None, Z, one, one, mean, one, 1, 0.0, mask, 0.0, one, one,
                                      dsum, None)
    assert bwd(dY=None) == hb.EINVAL and bwd(Z=one, mean=None) == hb.EINVAL and bwd(mask=one) == hb.EINVAL and bwd(dsum=one) == hb.EINVAL
    assert bwd(dY=off) == hb.EUNSUPPORTED and bwd(M=33) == hb.EUNSUPPORTED and bwd(Fy=9) == hb.EUNSUPPORTED
