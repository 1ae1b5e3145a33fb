"""The fp32 products as sums of bf16 products (k=1 convolution, forward and both gradients): tiles of both sizes, pieces
that straddle a row's end, and values that have no split -- infinities, NaN, magnitudes near the largest and below 2^-100
down to fp32's smallest, which go through the fp32 matrix instruction.

Reference: float64 products of the same values.  Bound per element, in units of 2^-24 sum|a||b|: a matrix instruction adds
sixteen products to its accumulator and rounds or truncates once (2 units per 16 k, as much again for the sums inside it),
and 8 for the parts left out, the two accumulators' sum and the sum of the split reductions: K / 4 + 8.  (The fp32
instruction, which takes two k at a time, stays below K.)"""
import numpy as np
import pytest
import torch

from util import conv_strides, dev, host

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


def run(hb, B, Nb, Ci, Co, L, x, w, dy):
    X, W, dY = dev(x, "f32"), dev(w, "f32"), dev(dy, "f32")
    Y, dX = torch.full((Nb, B * Co, L), float("nan"), device="cuda"), torch.full((Nb, B * Ci, L), float("nan"), device="cuda")
    dW = torch.full((B * Co, Ci), float("nan"), device="cuda")
    ws = torch.empty(hb.conv1x1_bwd_workspace_bytes(B, Nb, Ci, Co, L, 0) + 256, dtype=torch.uint8, device="cuda")
    ws = ws[-ws.data_ptr() % 256:]
    xs, ys = conv_strides(B, Ci, L), conv_strides(B, Co, L)
    hb.conv1x1_fwd(B, Nb, Ci, Co, L, 0, X, xs, W, None, Y, ys)
    hb.conv1x1_bwd(B, Nb, Ci, Co, L, 0, X, xs, W, dY, ys, dX, xs, dW, None, workspace=ws)
    x4, w3, d4 = (np.asarray(a, np.float64).reshape(s) for a, s in
                  ((x, (Nb, B, Ci, L)), (w, (B, Co, Ci)), (dy, (Nb, B, Co, L))))
    wt, xt = w3.transpose(0, 2, 1), x4.transpose(0, 1, 3, 2)
    with np.errstate(all="ignore"):
        refs = ((w3 @ x4, np.abs(w3) @ np.abs(x4), Ci), (wt @ d4, np.abs(wt) @ np.abs(d4), Co),
                ((d4 @ xt).sum(0), (np.abs(d4) @ np.abs(xt)).sum(0), Nb * L))
    return [(n, host(g).reshape(r.shape), r, m, k) for n, g, (r, m, k) in zip(("Y", "dX", "dW"), (Y, dX, dW), refs)]


def check(name, got, ref, mag, K, units=None):
    with np.errstate(all="ignore"):
        over = np.abs(ref) > 3.4e38                            # beyond fp32
        fin = np.isfinite(ref) & ~over
        assert np.array_equal(np.isnan(got), np.isnan(ref)), name
        assert np.array_equal(got[~fin & ~np.isnan(ref)], np.sign(ref[~fin & ~np.isnan(ref)]) * np.inf), name
        d, lim = np.abs(got - ref)[fin], (units or K / 4 + 8) * U * mag[fin] + 2.0 ** -126
    assert (d <= lim).all(), (name, float((d / lim).max()))


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [
    (2, 16, 72, 132, 1028),      # 128 x 128 tiles with remainders in every dimension, whole pieces
    (2, 16, 70, 130, 1030),      # the same, pieces that straddle the rows' ends
    (1, 3, 128, 65, 333),        # 64 x 64 tiles, odd everywhere
    (1, 2, 96, 68, 64),          # whole pieces, three k-tiles
    (1, 1, 65, 33, 4),           # one k past two tiles; a row of one piece
    (2, 2, 64, 64, 100),         # a reduction the fp32 instruction keeps
    (1, 2, 3, 70, 130),          # too few elements for a piece
    (1, 3, 201, 150, 333),       # straddling pieces in small tiles, enough k a workgroup for the split
    (1, 40, 22, 26, 1029),       # the same for the weight gradient
    (2, 20, 16, 130, 1500),      # 128 x 128 tiles of at most 16 k: the fp32 instruction's
    (2, 20, 14, 130, 1501),      # and with pieces that straddle
    (2, 5, 40, 48, 44),          # small tiles whose second k-tile is half empty
])
def test_products(hb, B, Nb, Ci, Co, L):
    r = np.random.default_rng(L)
    x, w, dy = (r.standard_normal(s).astype(np.float32) for s in ((Nb, B * Ci, L), (B * Co, Ci), (Nb, B * Co, L)))
    short = lambda K: K if K <= 64 or Ci < 4 else K / 4 + 8
    for n, got, ref, mag, K in run(hb, B, Nb, Ci, Co, L, x, w, dy):
        check(n, got, ref, mag, K, max(short(K), 4))


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(2, 16, 72, 132, 1028), (1, 2, 131, 67, 133)])
@pytest.mark.parametrize("what", ["inf", "nan", "largest", "small", "tiny", "subnormal", "subnormal among ordinary"])
def test_values_without_a_split(hb, B, Nb, Ci, Co, L, what):
    r = np.random.default_rng(7)
    x, w, dy = (r.standard_normal(s).astype(np.float32) for s in ((Nb, B * Ci, L), (B * Co, Ci), (Nb, B * Co, L)))
    if what in ("inf", "nan"):
        v = np.float32(what)
        x[1, 5, 17] = v
        x[0, Ci - 1, L - 1] = -v
        dy[1, 2, 3] = v
    elif what == "largest":                                    # rounds up to infinity in bf16; products within range
        x[1, 5, 17] = np.float32(3.402e38)
        dy[1, 2, 3] = np.float32(-3.402e38)
        w *= np.float32(2.0 ** -6)
    elif what == "small":                                      # tiny values among ordinary ones
        x[:, :, ::3] *= np.float32(2.0 ** -118)
        dy[:, :, ::3] *= np.float32(2.0 ** -118)
    elif what.startswith("subnormal"):                         # below bf16's smallest: the first part rounds to zero
        part = slice(None) if what == "subnormal" else slice(None, None, 3)
        x[:, :, part] *= np.float32(2.0 ** -140)
        dy[:, :, part] *= np.float32(2.0 ** -140)
        w *= np.float32(2.0 ** 100)
    else:                                                      # and nothing else: results near fp32's smallest normal numbers
        x *= np.float32(2.0 ** -118)
        dy *= np.float32(2.0 ** -118)
    for n, got, ref, mag, K in run(hb, B, Nb, Ci, Co, L, x, w, dy):
        if what in ("tiny", "subnormal") and n == "dW":
            continue                                           # 2^-236, 2^-280: below fp32
        if what == "largest" and n == "dW":
            assert not np.isnan(got).any()                     # products beyond fp32 may go either way at its edge
            continue
        check(n, got, ref, mag, K, max(K, 8))                  # the fp32 instruction's bound


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(1, 2, 128, 256, 256), (1, 1, 4096, 256, 256), (8, 2, 1024, 1024, 2500)])
def test_sums_of_one_sign(hb, B, Nb, Ci, Co, L):
    """Positive values throughout: partial sums grow with k, and an accumulation that rounds one way would be off by K / 16 half
    units.  One rounding to nearest per 16 k of partial sums up to the result, taken as independent, is 2^-24 sqrt(K / 16) at
    most in the 2-norm, and one unit more for the rest.  (The last weight gradient is one sum of 5000 products.)"""
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci)
    X, W, dY = (torch.rand(s, generator=g, device="cuda") for s in ((Nb, B, Ci, L), (B, Co, Ci), (Nb, B, Co, L)))
    Y, dX, dW = torch.empty_like(dY), torch.empty_like(X), torch.empty_like(W)
    ws = torch.empty(hb.conv1x1_bwd_workspace_bytes(B, Nb, Ci, Co, L, 0) + 256, dtype=torch.uint8, device="cuda")
    xs, ys = conv_strides(B, Ci, L), conv_strides(B, Co, L)
    hb.conv1x1_fwd(B, Nb, Ci, Co, L, 0, X, xs, W, None, Y, ys)
    hb.conv1x1_bwd(B, Nb, Ci, Co, L, 0, X, xs, W, dY, ys, dX, xs, dW, None, workspace=ws)
    x, w, d = X[:, B - 1].double(), W[B - 1].double(), dY[:, B - 1].double()
    ref_w = sum(d[n] @ x[n].t().contiguous() for n in range(Nb))
    for got, ref, K in ((Y[0, B - 1], w @ x[0], Ci), (dX[0, B - 1], w.t().contiguous() @ d[0], Co), (dW[B - 1], ref_w, Nb * L)):
        err = float((got.double() - ref).norm() / ref.norm())
        assert err <= U * (1 + (K / 16) ** 0.5), (K, err)


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(2, 4, 128, 1024, 256), (3, 5, 70, 601, 130), (1, 1, 3, 513, 5), (2, 64, 20, 512, 60), (1, 2, 64, 2050, 67)])
def test_data_gradient_of_few_tiles(hb, B, Nb, Ci, Co, L):
    """Few tiles under a long reduction: split with the workspace, whole without and for a dX with gaps; no further off float64 than
    whole, up to one rounding of the result."""
    g = torch.Generator(device="cuda")
    g.manual_seed(Co)
    W, dY = (torch.randn(s, generator=g, device="cuda") for s in ((B, Co, Ci), (Nb, B, Co, L)))
    ws = torch.empty(hb.conv1x1_bwd_workspace_bytes(B, Nb, Ci, Co, L, 0), dtype=torch.uint8, device="cuda")
    xs, ys = conv_strides(B, Ci, L), conv_strides(B, Co, L)
    got = []
    for gap, work in ((0, ws), (0, None), (0, ws[:64]), (8, ws)):
        out = torch.full((Nb, B, Ci, L + gap), float("nan"), device="cuda")
        st = (Ci * (L + gap), B * Ci * (L + gap), L + gap, 1) if gap else xs
        hb.conv1x1_bwd(B, Nb, Ci, Co, L, 0, None, None, W, dY, ys, out, st, None, None, workspace=work)
        assert not gap or torch.isnan(out[..., L:]).all()
        got.append(out[..., :L].contiguous())
    assert torch.equal(got[1], got[2]) and torch.equal(got[1], got[3])
    ref = torch.matmul(W.double().transpose(1, 2).contiguous(), dY.double())
    e = [((v.double() - ref).norm() / ref.norm()).item() for v in got[:2]]
    print(e)
    assert not torch.equal(got[0], got[1])
    assert e[0] <= e[1] + U / 2, e
