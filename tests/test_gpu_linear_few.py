"""Linear layers of few rows with the operators beside them: the bits of the single operators, at tile edges and remainders."""
import ctypes as C

import pytest
import torch

from paper_2102_02344_amd import binding as hb

DEV = "cuda"
TDT = {hb.F32: torch.float32, hb.BF16: torch.bfloat16}


def _rand(g, dt, *shape, scale=1.0):
    return ((torch.rand(shape, generator=g) * 2 - 1) * scale).to(TDT[dt]).to(DEV)


def _f32(g, *shape):
    return (torch.rand(shape, generator=g) + 0.5).to(DEV)


def _same(a, b, what):
    kind = torch.int32 if a.dtype == torch.float32 else torch.int16
    assert torch.equal(a.view(kind), b.view(kind)), what


BF16_SHAPES = [(1, 1, 8, 8), (2, 2, 96, 16), (3, 13, 1024, 512), (16, 16, 1216, 40), (5, 17, 72, 264), (8, 32, 512, 256), (40, 31, 136, 72)]
F32_SHAPES = [(1, 1, 4, 4), (2, 4, 1024, 256), (2, 4, 256, 16), (4, 32, 1024, 512), (4, 32, 512, 256), (3, 13, 68, 68), (5, 17, 100, 260), (9, 31, 36, 300),
              (1, 16, 64, 1028)]
SHAPES = [(hb.BF16,) + s for s in BF16_SHAPES] + [(hb.F32,) + s for s in F32_SHAPES]


def _linear(B, M, Fx, Fy, dt, x, w, bias, y, act=hb.ACT_NONE):
    """The split product and the sum of its parts as two launches (the entry point without a workspace keeps them)."""
    hb.linear_fwd_static(B, M, Fx, Fy, dt, x, w, bias, y, act)


@pytest.mark.gpu
@pytest.mark.parametrize("dt,B,M,Fx,Fy", SHAPES)
@pytest.mark.parametrize("drop", [False, True])
def test_linear_batchnorm(dt, B, M, Fx, Fy, drop):
    g = torch.Generator().manual_seed(B * 1000 + M)
    assert hb.linear_few_supported(B, M, Fx, Fy, dt)
    x, w, bias = _rand(g, dt, B, M, Fx), _rand(g, dt, B, Fx, Fy, scale=Fx ** -0.5), _rand(g, dt, B, Fy)
    gamma, beta = _f32(g, B, Fy), _f32(g, B, Fy) - 1.0
    mask = (torch.rand((B, M, Fy), generator=g) < 0.7).to(torch.uint8).to(DEV) if drop else None
    ls = (M * Fy, Fy, 1, 1)
    T = dict(dtype=TDT[dt], device=DEV)

    def outputs():
        return dict(z=torch.empty(B, M, Fy, **T), y=torch.empty(B, M, Fy, **T), yd=torch.empty(B, M, Fy, **T)), \
            dict(rm=torch.full((B, Fy), 0.25, device=DEV), rv=torch.full((B, Fy), 1.5, device=DEV),
                 mean=torch.empty(B, Fy, device=DEV), invstd=torch.empty(B, Fy, device=DEV))

    (o1, s1), (o2, s2) = outputs(), outputs()
    _linear(B, M, Fx, Fy, dt, x, w, bias, o1["z"])
    hb.bn_fwd(B, M, Fy, 1, dt, o1["z"], ls, gamma, beta, 1e-5, 0.1, s1["rm"], s1["rv"], s1["mean"], s1["invstd"], o1["y"], ls,
              hb.ACT_RELU)
    if drop:
        hb.dropout(B * M * Fy, dt, o1["y"], mask, 0.3, o1["yd"])
    hb.linear_bn_fwd(B, M, Fx, Fy, dt, x, w, bias, gamma, beta, 1e-5, 0.1, s2["rm"], s2["rv"], s2["mean"], s2["invstd"], o2["z"],
                     o2["y"], hb.ACT_RELU, 0.0, mask, 0.3 if drop else 0.0, o2["yd"] if drop else None)
    for k in ("z", "y") + (("yd",) if drop else ()):
        _same(o1[k], o2[k], k)
    for k in s1:
        _same(s1[k], s2[k], k)
    ws = torch.empty(max(4, hb.linear_fwd_workspace_bytes(B, M, Fx, Fy, dt)), dtype=torch.uint8, device=DEV)
    for act in (hb.ACT_NONE, hb.ACT_RELU):
        _linear(B, M, Fx, Fy, dt, x, w, bias, o1["y"], act)
        hb.linear_fwd_ws(B, M, Fx, Fy, dt, x, w, bias, o2["y"], act, workspace=ws)
        _same(o1["y"], o2["y"], ("forward", act))

    # backward: this Linear's gradients, and on through a BatchNorm or a ReLU below it (of Fx channels)
    dy, zb = _rand(g, dt, B, M, Fy, scale=0.1), _rand(g, dt, B, M, Fx)
    gb, bb = _f32(g, B, Fx), _f32(g, B, Fx) - 1.0
    mean, invstd = zb.float().mean(1).contiguous(), _f32(g, B, Fx)
    maskb = (torch.rand((B, M, Fx), generator=g) < 0.7).to(torch.uint8).to(DEV) if drop else None
    lx = (M * Fx, Fx, 1, 1)
    wb = torch.empty(max(4, hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, dt)), dtype=torch.uint8, device=DEV)
    dx, dd, dz, da = (torch.empty(B, M, Fx, **T) for _ in range(4))
    dw, db = torch.empty(B, Fx, Fy, device=DEV), torch.empty(B, Fy, device=DEV)
    sums = [torch.empty(B, Fx, device=DEV) for _ in range(3)]
    hb.linear_bwd(B, M, Fx, Fy, dt, x, w, dy, dx, dw, db, wb)
    if drop:
        hb.dropout(B * M * Fx, dt, dx, maskb, 0.3, dd)
    hb.bn_bwd(B, M, Fx, 1, dt, zb, lx, dd if drop else dx, lx, gb, bb, mean, invstd, dz, lx, sums[0], sums[1], hb.ACT_RELU, 0.0, sums[2])
    hb.act_bwd(B * M * Fx, dt, zb, dd if drop else dx, da, hb.ACT_RELU, 0.0, 1)
    dx2, dz2, da2 = (torch.empty(B, M, Fx, **T) for _ in range(3))
    dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
    dw3, dw4 = torch.empty_like(dw), torch.empty_like(dw)
    sums2 = [torch.empty(B, Fx, device=DEV) for _ in range(3)]
    p = 0.3 if drop else 0.0
    hb.linear_bwd_bn(B, M, Fx, Fy, dt, x, w, dy, dx2, dw2, db2)
    hb.linear_bwd_bn(B, M, Fx, Fy, dt, x, w, dy, dz2, dw3, None, zb, gb, bb, mean, invstd, hb.ACT_RELU, 0.0, maskb, p, *sums2)
    hb.linear_bwd_act(B, M, Fx, Fy, dt, x, w, dy, da2, dw4, None, zb, hb.ACT_RELU, 0.0, maskb, p)
    for a, b, what in ((dx, dx2, "dX"), (dw, dw2, "dW"), (dw, dw3, "dW"), (dw, dw4, "dW"), (db, db2, "dbias"), (dz, dz2, "dZ"),
                       (da, da2, "through the ReLU")):
        _same(a, b, what)
    for a, b, what in zip(sums, sums2, ("dgamma", "dbeta", "sum of dZ")):
        _same(a, b, what)


@pytest.mark.gpu
@pytest.mark.parametrize("dt,B,M,Fx,K", [(hb.BF16, 1, 1, 8, 8), (hb.BF16, 3, 13, 256, 16), (hb.BF16, 8, 32, 256, 16), (hb.BF16, 2, 17, 1000, 32),
                                         (hb.F32, 2, 4, 256, 16), (hb.F32, 1, 1, 4, 4), (hb.F32, 3, 31, 100, 28)])
def test_linear_cross_entropy(dt, B, M, Fx, K):
    g = torch.Generator().manual_seed(M)
    x, w, bias = _rand(g, dt, B, M, Fx), _rand(g, dt, B, Fx, K, scale=3 * Fx ** -0.5), _rand(g, dt, B, K)
    labels = torch.randint(K, (B, M), generator=g, dtype=torch.int32).to(DEV)
    z1, z2, d1, d2 = (torch.empty(B, M, K, dtype=TDT[dt], device=DEV) for _ in range(4))
    l1, l2 = torch.empty(B, device=DEV), torch.empty(B, device=DEV)
    _linear(B, M, Fx, K, dt, x, w, bias, z1)
    hb.softmax_xent(B, M, K, dt, z1, labels, l1, d1)
    hb.linear_xent(B, M, Fx, K, dt, x, w, bias, z2, labels, l2, d2)
    for a, b, what in ((z1, z2, "logits"), (l1, l2, "loss"), (d1, d2, "dlogits")):
        _same(a, b, what)


@pytest.mark.gpu
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 1e-38, 1e-42, -3.39e38])
def test_values_without_a_split(value):
    """Such a value in dY: the data gradient of every column takes the fp32 instruction, as the product's tile does."""
    B, M, Fx, Fy = 2, 20, 96, 128
    g = torch.Generator().manual_seed(7)
    x, w, dy = _rand(g, hb.F32, B, M, Fx), _rand(g, hb.F32, B, Fx, Fy), _rand(g, hb.F32, B, M, Fy)
    dy[1, 3, 100] = value
    dx, dx2 = torch.empty(B, M, Fx, device=DEV), torch.empty(B, M, Fx, device=DEV)
    dw, dw2 = torch.empty(B, Fx, Fy, device=DEV), torch.empty(B, Fx, Fy, device=DEV)
    wb = torch.empty(max(4, hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.F32)), dtype=torch.uint8, device=DEV)
    hb.linear_bwd(B, M, Fx, Fy, hb.F32, x, w, dy, dx, dw, None, wb)
    hb.linear_bwd_bn(B, M, Fx, Fy, hb.F32, x, w, dy, dx2, dw2, None)
    for a, b in ((dx, dx2), (dw, dw2)):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num())


def test_what_is_declined():
    ok = lambda *a: hb.linear_few_supported(*a)
    assert ok(8, 32, 1024, 512, hb.BF16) and ok(1, 1, 8, 8, hb.BF16) and ok(4, 32, 1024, 512, hb.F32) and ok(1, 1, 4, 4, hb.F32)
    assert not ok(8, 33, 1024, 512, hb.BF16) and not ok(8, 33, 1024, 512, hb.F32)
    assert not ok(8, 32, 1028, 512, hb.BF16) and not ok(8, 32, 256, 9, hb.BF16) and not ok(16, 32, 1224, 512, hb.BF16) and not ok(1, 32, 1216, 40, hb.BF16)
    assert not ok(4, 32, 1022, 512, hb.F32) and not ok(4, 32, 256, 10, hb.F32) and not ok(16, 16, 1216, 40, hb.F32)   # 76 k a piece
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

    def bwd_act(H=one, dY=one, mask=None, p=0.0, act=1):
        return raw.hfta_linear_bwd_act(8, 32, 256, 64, 0, one, one, dY, one, one, None, H, act, 0.0, mask, p, None)
    assert bwd_act(H=None) == hb.EINVAL and bwd_act(dY=None) == hb.EINVAL and bwd_act(mask=one, p=1.0) == hb.EINVAL
    assert bwd_act(dY=off) == hb.EUNSUPPORTED and bwd_act(act=hb.ACT_GELU) == hb.EUNSUPPORTED


def test_more_channels_than_an_int_counts():
    """A channel of a model is numbered in 32 bits."""
    raw, one = hb.raw(), C.c_void_p(256)
    for Fx, Fy in ((8, 32776), (32776, 8)):
        assert not hb.linear_few_supported(65535, 32, Fx, Fy, hb.BF16)
        rc = raw.hfta_linear_bwd_bn(65535, 32, Fx, Fy, hb.BF16, one, one, one, one, one, None, one, one, one, one, one, 1, 0.0, None, 0.0, one, one,
                                    None, None)
        assert rc == hb.EUNSUPPORTED


@pytest.mark.gpu
@pytest.mark.parametrize("B,M", [(16, 32), (16, 17), (16, 16), (15, 32)])
def test_fp32_weight_gradient_of_many_tiles(B, M):
    """From 512 tiles of 128 x 128 outputs on and 17 rows on the single operator takes the product of three bf16 parts: declined here."""
    Fx, Fy = 1024, 512
    g = torch.Generator().manual_seed(B + M)
    x, w, dy = _rand(g, hb.F32, B, M, Fx), _rand(g, hb.F32, B, Fx, Fy), _rand(g, hb.F32, B, M, Fy)
    dx, dx2, dw, dw2, da = (torch.full(s, float("nan"), device=DEV) for s in ((B, M, Fx), (B, M, Fx), (B, Fx, Fy), (B, Fx, Fy), (B, M, Fx)))
    wb = torch.empty(max(4, hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.F32)), dtype=torch.uint8, device=DEV)
    hb.linear_bwd(B, M, Fx, Fy, hb.F32, x, w, dy, dx, dw, None, wb)
    if B == 16 and M > 16:
        for call in (lambda: hb.linear_bwd_bn(B, M, Fx, Fy, hb.F32, x, w, dy, dx2, dw2, None),
                     lambda: hb.linear_bwd_act(B, M, Fx, Fy, hb.F32, x, w, dy, da, dw2, None, x)):
            with pytest.raises(hb.HftaError) as e:
                call()
            assert e.value.status == hb.EUNSUPPORTED
        assert torch.isnan(dx2).all() and torch.isnan(dw2).all() and not hb.linear_few_supported(B, M, Fx, Fy, hb.F32)
    else:
        hb.linear_bwd_bn(B, M, Fx, Fy, hb.F32, x, w, dy, dx2, dw2, None)
        _same(dx, dx2, "dX")
        _same(dw, dw2, "dW")


def test_where_one_launch_is_the_sooner_way():
    """Both sides of the lines: k of a wavefront times workgroups of the forward, workgroups of the backward, LDS in fp32."""
    ok = hb.linear_few_supported
    assert ok(32, 32, 1024, 512, hb.BF16) and not ok(33, 32, 1024, 512, hb.BF16) and not ok(64, 4, 1024, 512, hb.BF16)
    assert ok(96, 32, 512, 256, hb.BF16) and not ok(97, 32, 512, 256, hb.BF16) and not ok(256, 13, 512, 256, hb.BF16)
    assert ok(307, 32, 256, 16, hb.BF16) and not ok(308, 32, 256, 16, hb.BF16)
    assert ok(64, 32, 256, 16, hb.F32) and not ok(65, 32, 256, 16, hb.F32) and not ok(512, 4, 64, 64, hb.F32)
    assert ok(51, 4, 64, 320, hb.F32) and not ok(52, 4, 64, 320, hb.F32)


@pytest.mark.gpu
@pytest.mark.parametrize("dt,B,M,Fx,Fy", [(hb.BF16, 65, 32, 1024, 512), (hb.BF16, 300, 3, 88, 136), (hb.BF16, 24, 32, 1024, 512),
                                          (hb.BF16, 25, 32, 1024, 512), (hb.F32, 300, 5, 64, 64), (hb.F32, 2, 4, 1024, 512), (hb.F32, 4, 4, 1024, 512)])
def test_beyond_those_lines(dt, B, M, Fx, Fy):
    """The calls take such shapes and leave the same bits; so does the forward with a workspace on either of its routes."""
    g = torch.Generator().manual_seed(B)
    x, w, bias, gamma, beta = _rand(g, dt, B, M, Fx), _rand(g, dt, B, Fx, Fy, scale=Fx ** -0.5), _rand(g, dt, B, Fy), _f32(g, B, Fy), _f32(g, B, Fy)
    z, z2, z3, y, y2 = (torch.empty(B, M, Fy, dtype=TDT[dt], device=DEV) for _ in range(5))
    ls = (M * Fy, Fy, 1, 1)
    s1, s2 = ([torch.ones(B, Fy, device=DEV) for _ in range(4)] for _ in range(2))
    ws = torch.empty(max(4, hb.linear_fwd_workspace_bytes(B, M, Fx, Fy, dt)), dtype=torch.uint8, device=DEV)
    if hb.linear_fwd_workspace_bytes(B, M, Fx, Fy, dt) <= hb.linear_fwd_static_max_bytes():
        _linear(B, M, Fx, Fy, dt, x, w, bias, z)
    else:
        hb.linear_fwd_ws(B, M, Fx, Fy, dt, x, w, bias, z, workspace=ws)
    hb.bn_fwd(B, M, Fy, 1, dt, z, ls, gamma, beta, 1e-5, 0.1, *s1, y, ls, hb.ACT_RELU)
    hb.linear_bn_fwd(B, M, Fx, Fy, dt, x, w, bias, gamma, beta, 1e-5, 0.1, *s2, z2, y2, hb.ACT_RELU)
    hb.linear_fwd_ws(B, M, Fx, Fy, dt, x, w, bias, z3, workspace=ws)
    for a, b, what in [(z, z2, "z"), (z, z3, "with a workspace"), (y, y2, "y")] + [(a, b, "statistics") for a, b in zip(s1, s2)]:
        _same(a, b, what)
    dy, dx, dx2 = _rand(g, dt, B, M, Fy, scale=0.1), torch.empty_like(x), torch.empty_like(x)
    dw, dw2, db, db2 = torch.empty(B, Fx, Fy, device=DEV), torch.empty(B, Fx, Fy, device=DEV), torch.empty(B, Fy, device=DEV), torch.empty(B, Fy, device=DEV)
    wb = torch.empty(max(4, hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, dt)), dtype=torch.uint8, device=DEV)
    hb.linear_bwd(B, M, Fx, Fy, dt, x, w, dy, dx, dw, db, wb)
    hb.linear_bwd_bn(B, M, Fx, Fy, dt, x, w, dy, dx2, dw2, db2)
    for a, b, what in ((dx, dx2, "dX"), (dw, dw2, "dW"), (db, db2, "dbias")):
        _same(a, b, what)


# heads of which the first layer, the last, or those in between take the one-launch calls
@pytest.mark.gpu
@pytest.mark.parametrize("net,dt,B", [("cls", "bf16", 40), ("cls", "f32", 16), ("cls", "bf16", 8), ("clst", "bf16", 9), ("clst", "f32", 9)])
def test_arrays_either_way(net, dt, B, monkeypatch):
    """A step of an array whose head takes the one-launch calls layer by layer has the bits of one that makes the single calls."""
    import hfta_inputs as hi
    from paper_2102_02344_amd import arrays
    if net == "cls":
        spec = hi.spec_c1(B=B, Nb=4, L=64, dtype=dt)
        inp, make, fc = hi.pointnet_cls_inputs(spec), arrays.FusedPointNetCls, spec.fc
    else:
        spec = hi.PointNetTSpec(cls=hi.spec_c1(B=B, Nb=4, L=64, dtype=dt))
        inp, make, fc = hi.pointnet_t_inputs(spec), arrays.FusedPointNetClsT, (1024, 512, 256, 64 * 64)
    code = hb.BF16 if dt == "bf16" else hb.F32
    takes = [bool(hb.linear_few_supported(B, 4, a, b, code)) for a, b in zip(fc, fc[1:])]
    print(net, dt, B, takes, flush=True)
    assert any(takes) and (B == 8 or not all(takes))
    got = []
    for route in ("as it is", "single"):
        if route == "single":
            monkeypatch.setattr(arrays.hb, "linear_few_supported", lambda *a: False)
        a = make(spec, inp)
        a.forward_backward()
        got.append([a.loss.clone(), a.grad.clone()] + [v.clone() for v in a.running.values()] + [v.clone() for v in a.saved.values()])
    for x, y in zip(*got):
        _same(x.contiguous().view(-1), y.contiguous().view(-1), (net, tuple(x.shape)))
