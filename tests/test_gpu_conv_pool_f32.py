"""The fp32 pair that keeps the convolution's output out of memory: the forward against hfta_conv1x1_bn_pool_fwd, bit for bit,
the backward against float64 and against the chain of stored operators."""
import pytest
import torch

from util import conv_strides

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


def reference(X, W, bias, gam, bet, idx, dV, act, slope, eps=1e-5):
    """dX, dW, dgamma, dbeta in float64; X [Nb, B, Ci, L]."""
    Nb, B, Ci, L = X.shape
    Co, out = W.shape[1], ([], [], [], [])
    for b in range(B):
        x, w = X[:, b].double(), W[b].double()
        z = torch.matmul(w, x) + bias[b].double()[:, None]
        mu, iv = z.mean((0, 2))[:, None], (z.var((0, 2), unbiased=False) + eps).rsqrt()[:, None]
        xh = (z - mu) * iv
        g, bt = gam[b].double()[:, None], bet[b].double()[:, None]
        ix = idx[b].long().unsqueeze(-1)
        hit = xh.gather(2, ix)
        pre = hit * g + bt
        gr = dV[b].double().unsqueeze(-1) * torch.where(pre > 0, 1.0, 1.0 if act == 0 else slope if act == 2 else 0.0)
        dbt, dg, m = gr.sum((0, 2)), (gr * hit).sum((0, 2)), Nb * L
        dz = g * iv * (torch.zeros_like(z).scatter_(2, ix, gr) - dbt[:, None] / m - xh * dg[:, None] / m)
        out[0].append(torch.matmul(w.t().contiguous(), dz))
        out[1].append(sum(torch.matmul(dz[n], x[n].t().contiguous()) for n in range(Nb)))
        out[2].append(dg)
        out[3].append(dbt)
    return torch.stack(out[0], 1), torch.stack(out[1]), torch.stack(out[2]), torch.stack(out[3])


def both_ways(hb, dims, X, W, bias, gam, bet, dV, act, slope):
    """Forward results and (dX, dW, dgamma, dbeta) of the chain of stored operators and of the pair."""
    B, Nb, Ci, Co, L = dims
    xs, zs, vs = conv_strides(B, Ci, L), conv_strides(B, Co, L), (Nb * Co, Co, 1)
    need = hb.conv1x1_bn_maxpool_f32_workspace_bytes(*dims)
    assert need > 0
    ws = torch.empty(max(need, hb.conv1x1_bwd_workspace_bytes(*dims, 0)), dtype=torch.uint8, device="cuda")
    e = lambda *s: torch.full(s, float("nan"), device="cuda")
    res = []
    for stored in (True, False):
        o = dict(mean=e(B * Co), invstd=e(B * Co), V=e(B, Nb, Co), idx=torch.full((B, Nb, Co), -1, dtype=torch.int32, device="cuda"),
                 rm=torch.zeros(B * Co, device="cuda"), rv=torch.ones(B * Co, device="cuda"))
        bn = (W, bias, gam, bet, 1e-5, 0.1, o["rm"], o["rv"], o["mean"], o["invstd"])
        dX, dW, db, dg, dbt = e(Nb, B, Ci, L), e(B, Co, Ci), e(B, Co), e(B, Co), e(B, Co)
        if stored:
            Z, dZ = e(Nb, B * Co, L), e(Nb, B * Co, L)
            hb.conv1x1_bn_pool_fwd(*dims, 0, X, xs, *bn, Z, zs, None, None, o["V"], o["idx"], vs, act, slope, ws)
            hb.bn_bwd_maxpool(B, Nb, Co, L, 0, Z, zs, dV, o["idx"], vs, gam, bet, o["mean"], o["invstd"], dZ, zs, dg, dbt, act, slope, db)
            hb.conv1x1_bwd(*dims, 0, X, xs, W, dZ, zs, dX, xs, dW, None, ws)
            del Z, dZ
        else:
            zhit = e(B, Nb, Co)
            hb.conv1x1_bn_maxpool_f32_fwd(*dims, X, xs, *bn, o["V"], o["idx"], vs, zhit, act, slope, ws)
            hb.conv1x1_bn_maxpool_f32_bwd(*dims, X, xs, W, bias, zhit, dV, o["idx"], vs, gam, bet, o["mean"], o["invstd"], dX, xs, dW, db,
                                          dg, dbt, act, slope, ws)
            assert not db.any()
        res.append((o, (dX, dW, dg, dbt)))
    return res


@pytest.mark.parametrize("dims,act,slope,shift", [((3, 29, 128, 1024, 1023), 1, 0.0, 0.0), ((8, 64, 68, 70, 130), 1, 0.0, 2.0),
                                                  ((2, 32, 96, 200, 1030), 2, 0.2, 0.0), ((1, 512, 128, 65, 128), 0, 0.0, 0.0),
                                                  ((2, 32, 100, 513, 1028), 1, 0.0, 10.0)])
def test_pair(hb, dims, act, slope, shift):
    B, Nb, Ci, Co, L = dims
    print(f"fp32 tail {dims} act={act} shift={shift}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    X = torch.relu(r(Nb, B, Ci, L)) + shift
    X[:, :, :, L // 2] *= 3.0                                # a point that many channels choose: more hits than a wavefront
    W, bias, gam, bet, dV = r(B, Co, Ci) * (2.0 / Ci) ** 0.5, 0.1 * r(B, Co), 1.0 + 0.2 * r(B, Co), 0.3 * r(B, Co), r(B, Nb, Co)
    gam[:, ::7] *= -1.0
    gam[0, 3], bet[0, 3], bet[0, 5] = 0.0, 0.5, -50.0        # all points equal; all points clipped
    (a, ga), (b, gb) = both_ways(hb, dims, X, W, bias, gam, bet, dV, act, slope)
    same = torch.ones_like(a["V"], dtype=torch.bool)
    same[0, :, 3] = False                                    # gamma = 0: z at point 0 by another order of the sum
    for k in a:
        assert torch.equal(a[k][same], b[k][same]) if k == "V" else torch.equal(a[k], b[k]), k
    assert torch.allclose(a["V"], b["V"], rtol=1e-6, atol=0)
    # Sums of K <= 1024 products of fp32 values rounded to 2^-24 each: sqrt(K) 2^-24 = 2e-6 of their norm; and no further off
    # than the stored chain, whose rounding of 1e-7 in what cancels is the yardstick where the mean is large.
    for name, q, s, t in zip(("dX", "dW", "dgamma", "dbeta"), reference(X, W, bias, gam, bet, a["idx"], dV, act, slope), ga, gb):
        err = [((v.double() - q).norm() / q.norm()).item() for v in (s, t)]
        print(name, err)
        assert err[1] <= 2e-6 and err[1] <= 1.05 * err[0] + 2e-8, (name, err)


@pytest.mark.parametrize("where", ["w", "x", "both"])
@pytest.mark.parametrize("dims", [(4, 64, 68, 161, 129), (1, 300, 128, 1024, 160)])
def test_values_without_a_split(hb, dims, where):
    """Values below 2^-100 and infinities have no three bf16 parts: the tiles that hold them take the fp32 instruction, the others do
    not, and the forward's results are the stored form's, bit for bit."""
    B, Nb, Ci, Co, L = dims
    print(f"fp32 tail {dims} without a split in {where}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    X, W, gam = r(Nb, B, Ci, L), r(B, Co, Ci), r(B, Co)
    if where != "x":
        W[B - 1, Co - 1, 0], W[0, 40, Ci - 1] = 2.0 ** -110, -2.0 ** -120
    if where != "w":
        X[Nb - 1, 0, Ci - 1, L - 1], X[0, B - 1, 0, 3] = 2.0 ** -130, 2.0 ** -105
    if where == "both":
        W[0, 7, 2] = float("inf")
    (a, _), (b, _) = both_ways(hb, dims, X, W, r(B, Co), gam, r(B, Co), r(B, Nb, Co), 1, 0.0)
    for k in a:
        assert torch.equal(a[k].view(torch.int32)[..., 8:], b[k].view(torch.int32)[..., 8:]), k


def _padded(X):
    """Every cloud's first 96 points are one and the same, five spreads from the others."""
    X[:, :, :, :96] = X.mean((0, 3), keepdim=True) + 5.0 * X.std((0, 3), keepdim=True)


def _front(X):
    """The first cloud of each model lies three spreads from the others."""
    X[0] += 3.0 * X.std((0, 3), keepdim=True)[0]


def _ordered(X):
    """Clouds sorted along a direction that all channels see."""
    X += 2.0 * X[:, :, :1].sort(3).values


def _correlated(X):
    """Channels that are pairwise correlated at 0.99."""
    X.mul_(0.1).add_(0.99 ** 0.5 * torch.randn(X[:, :, :1].shape, generator=torch.Generator(device="cuda").manual_seed(4), device="cuda"))


@pytest.mark.parametrize("how", [_padded, _front, _ordered, _correlated])
@pytest.mark.parametrize("dims", [(2, 16, 128, 256, 2048), (3, 29, 68, 130, 1023), (64, 8, 68, 70, 2050), (64, 1, 72, 66, 16400)])
def test_points_that_are_not_alike(hb, dims, how):
    """dW of clouds whose points are not spread alike over their memory: no further off float64 than the stored chain is (see
    test_pair)."""
    print(f"fp32 tail {dims} {how.__name__}", flush=True)
    B, Nb, Ci, Co, L = dims
    gen = torch.Generator(device="cuda").manual_seed(9)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    X = r(Nb, B, Ci, L)
    how(X)
    W, bias, gam, bet, dV = r(B, Co, Ci) * (2.0 / Ci) ** 0.5, 0.1 * r(B, Co), 1.0 + 0.2 * r(B, Co), 0.3 * r(B, Co), r(B, Nb, Co)
    (a, ga), (_, gb) = both_ways(hb, dims, X, W, bias, gam, bet, dV, 1, 0.0)
    for name, q, s, t in zip(("dX", "dW", "dgamma", "dbeta"), reference(X, W, bias, gam, bet, a["idx"], dV, 1, 0.0), ga, gb):
        err = [((v.double() - q).norm() / q.norm()).item() for v in (s, t)]
        print(name, err)
        assert err[1] <= 2e-6 and err[1] <= 1.05 * err[0] + 2e-8, (name, err)


def test_refuses_and_array_route(hb):
    assert hb.conv1x1_bn_maxpool_f32_workspace_bytes(4, 32, 128, 1024, 2500) > 0
    for dims in ((4, 32, 64, 1024, 2500), (4, 32, 132, 1024, 2500), (4, 32, 128, 1028, 2500), (1, 4, 128, 1024, 256), (4, 32, 126, 1024, 2500),
                 (600, 1, 128, 128, 100)):
        assert hb.conv1x1_bn_maxpool_f32_workspace_bytes(*dims) == 0
    import hfta_inputs as hi
    from paper_2102_02344_amd.arrays import FusedPointNetCls
    spec = hi.spec_c1(B=2, Nb=16, L=2050, dtype="f32")
    inp = hi.pointnet_cls_inputs(spec)
    lean, stored = FusedPointNetCls(spec, inp), FusedPointNetCls(spec, inp, fused_tail=False)
    assert lean.tail_f32_ws > 0 and stored.tail_f32_ws == 0
    lean.forward_backward()
    stored.forward_backward()
    assert torch.equal(lean.pooled, stored.pooled) and torch.equal(lean.loss, stored.loss)
    for name, _ in lean.shapes:
        if name.startswith("fc") or name.endswith(("conv4.bn.g", "conv4.w")):
            x, y = lean.g(name).double(), stored.g(name).double()
            assert (x - y).norm() <= 4e-6 * y.norm() + 1e-12, name


def _per_point_gradients(arr, dpool):
    """Gradients of the per-point layers in float64 from the gradient of the pooled values, at the array's own argmax."""
    s, B, Nb, L = arr.spec, arr.B, arr.Nb, arr.L
    out = {}
    for b in range(B):
        x, par = arr.points.view(Nb, B, s.conv[0], L)[:, b].double(), {}
        for i, (ci, co) in enumerate(zip(s.conv[:-1], s.conv[1:])):
            k = f"conv{i}"
            for n, shape in ((".w", (co, ci)), (".b", (co, 1)), (".bn.g", (co, 1)), (".bn.b", (co, 1))):
                par[k + n] = arr.master(k + n).view(B, *shape)[b].double().requires_grad_()
            z = torch.matmul(par[k + ".w"], x) + par[k + ".b"]
            mu, var = z.mean((0, 2), keepdim=True), z.var((0, 2), unbiased=False, keepdim=True)
            x = torch.relu((z - mu) * (var + arr.BN_EPS).rsqrt() * par[k + ".bn.g"] + par[k + ".bn.b"])
        x.gather(2, arr.pool_idx[b].long().unsqueeze(-1)).squeeze(-1).backward(dpool[b].double())
        for n, v in par.items():
            out.setdefault(n, []).append(v.grad.reshape(-1))
    return {n: torch.stack(v) for n, v in out.items()}


def test_array_gradients_behind_the_tail():
    """A plain step's gradients below the tail are no further off float64 than those of the stored route (half as much again for the
    rounding of the layers below, which is another on each route); and a step that showed a probe every tensor leaves the next
    plain one as it was."""
    import hfta_inputs as hi
    from paper_2102_02344_amd.arrays import FusedPointNetCls
    spec = hi.spec_c1(B=2, Nb=16, L=2050, dtype="f32")
    inp = hi.pointnet_cls_inputs(spec)
    lean, stored = FusedPointNetCls(spec, inp), FusedPointNetCls(spec, inp, fused_tail=False)
    assert lean.tail_f32_ws > 0 and stored.tail_f32_ws == 0
    grads, kept = [], {}

    def probe(op, **t):
        if op == "linear_bwd" and t["layer"] == "fc0":
            kept["dpool"] = t["dx"].clone()
    for a, p in ((lean, None), (stored, probe)):
        a.forward_backward(p)
        grads.append({n: a.g(n).clone() for n, _ in a.shapes})
    assert torch.equal(lean.pool_idx, stored.pool_idx)
    ref = _per_point_gradients(stored, kept["dpool"].view(2, 16, -1))
    for n, q in ref.items():
        if n.endswith(".b") and not n.endswith(".bn.b"):
            continue                                       # in front of a BatchNorm: zero but for rounding
        err = [((g[n].double().reshape(q.shape) - q).norm() / q.norm()).item() for g in grads]
        print(n, err)
        assert err[0] <= 1.5 * err[1] + 1e-7, (n, err)
    lean.forward_backward(probe)
    lean.forward_backward()
    for n, _ in lean.shapes:
        assert torch.equal(lean.g(n), grads[0][n]), n


def test_workspace_without_the_weights_parts(hb):
    """A workspace that holds the partial sums and not W's parts beside them: the general product, the same results; less is refused."""
    B, Nb, Ci, Co, L = dims = (2, 14, 68, 1024, 4000)
    full, small = hb.conv1x1_bn_maxpool_f32_workspace_bytes(*dims), hb.conv1x1_bn_pool_fwd_workspace_bytes(*dims, 0)
    assert small < full
    gen = torch.Generator(device="cuda").manual_seed(2)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    X, W, bias, gam, bet, dV = r(Nb, B, Ci, L), 0.2 * r(B, Co, Ci), r(B, Co), r(B, Co), r(B, Co), r(B, Nb, Co)
    xs, vs = conv_strides(B, Ci, L), (Nb * Co, Co, 1)

    def run(size):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        e = lambda *s: torch.full(s, float("nan"), device="cuda")
        idx, stats = torch.full((B, Nb, Co), -1, dtype=torch.int32, device="cuda"), [torch.ones(B * Co, device="cuda") for _ in range(4)]
        V, zhit, dX, dW, dg, dbt = e(B, Nb, Co), e(B, Nb, Co), e(Nb, B, Ci, L), e(B, Co, Ci), e(B, Co), e(B, Co)
        hb.conv1x1_bn_maxpool_f32_fwd(*dims, X, xs, W, bias, gam, bet, 1e-5, 0.1, *stats, V, idx, vs, zhit, 1, 0.0, ws)
        hb.conv1x1_bn_maxpool_f32_bwd(*dims, X, xs, W, bias, zhit, dV, idx, vs, gam, bet, stats[2], stats[3], dX, xs, dW, None, dg, dbt, 1, 0.0, ws)
        return [V, idx, zhit, dX, dW, dg, dbt] + stats
    for a, b in zip(run(full), run(small)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    with pytest.raises(hb.HftaError):
        run(small - 256)


@pytest.mark.parametrize("value", [float("inf"), -float("inf"), float("nan")])
@pytest.mark.parametrize("dims", [(1, 520, 68, 161, 129), (2, 300, 128, 1024, 160)])
def test_channel_of_no_numbers(hb, dims, value):
    """A channel whose weights hold no number: its statistics, its values and the point it names (the first, and never one past the row,
    here in rows with a last tile of one and of 32 points) are those of the stored form, and the other channels do not notice."""
    B, Nb, Ci, Co, L = dims
    print(f"fp32 tail {dims} with {value}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(6)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    X, W, gam = r(Nb, B, Ci, L), r(B, Co, Ci), r(B, Co)
    W[0, 7, 2] = value
    W[B - 1, Co - 1, :] = value
    (a, _), (b, _) = both_ways(hb, dims, X, W, r(B, Co), gam, r(B, Co), r(B, Nb, Co), 1, 0.0)
    for k in a:
        v, w = a[k], b[k]
        assert torch.equal(torch.isnan(v), torch.isnan(w)) and torch.equal(v.nan_to_num(), w.nan_to_num()), k
    assert (b["idx"][0, :, 7] == 0).all() and (b["idx"][B - 1, :, Co - 1] == 0).all() and ((b["idx"] >= 0) & (b["idx"] < L)).all()
    assert torch.isnan(b["mean"].view(B, Co)[0, 7]) or torch.isinf(b["mean"].view(B, Co)[0, 7])
