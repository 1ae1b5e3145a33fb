"""k=1 convolutions whose rows are multiples of 8 bytes but not of 16 (an odd number of groups of four points), in sizes that the
256x256 product kernels take: the last piece of a row has four of its eight elements.  Rows lie apart in memory with NaN
between them, so that an element read past a row's end shows."""
import numpy as np
import pytest
import torch

from test_gpu_ops import f32_tol
from util import DT, TOL, check, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


def padded(gen, rows, L, pitch, scale=1.0):
    t = torch.full((rows, pitch), float("nan"), dtype=torch.bfloat16)
    t[:, :L] = torch.randn((rows, L), generator=gen) * scale
    return t.cuda(), t[:, :L].double()


@pytest.mark.parametrize("B,Nb,Ci,Co,L,pad", [(2, 40, 264, 516, 516, 4), (1, 33, 512, 776, 772, 8), (2, 24, 520, 260, 1028, 0)])
def test_forward_and_gradients(hb, B, Nb, Ci, Co, L, pad):
    print(f"rows of 8 bytes B={B} Nb={Nb} Ci={Ci} Co={Co} L={L} pad={pad}", flush=True)
    gen = torch.Generator().manual_seed(7)
    P, dt = L + pad, DT["bf16"]
    strides = lambda C: (C * P, B * C * P, P, 1)
    X, x = padded(gen, Nb * B * Ci, L, P)
    dY, dy = padded(gen, Nb * B * Co, L, P)
    W = (torch.randn((B, Co, Ci), generator=gen) / np.sqrt(Ci)).bfloat16()
    bias = torch.randn((B, Co), generator=gen).bfloat16()
    x, dy, w = x.view(Nb, B, Ci, L), dy.view(Nb, B, Co, L), W.double()
    Wd, Bd = W.cuda(), bias.cuda()
    ws = torch.empty(max(hb.conv1x1_bwd_workspace_bytes(B, Nb, Ci, Co, L, dt), 4), dtype=torch.uint8, device="cuda")

    Y = torch.zeros((Nb, B, Co, P), dtype=torch.bfloat16, device="cuda")
    hb.conv1x1_fwd(B, Nb, Ci, Co, L, dt, X, strides(Ci), Wd, Bd, Y, strides(Co))
    check(host(Y[..., :L]), (torch.matmul(w, x) + bias.double()[:, :, None]).numpy(), TOL["bf16"], "Y")
    assert not Y[..., L:].any()
    dX = torch.zeros((Nb, B, Ci, P), dtype=torch.bfloat16, device="cuda")
    hb.conv1x1_bwd(B, Nb, Ci, Co, L, dt, None, None, Wd, dY, strides(Co), dX, strides(Ci), None, None, ws)
    check(host(dX[..., :L]), torch.matmul(w.transpose(1, 2).contiguous(), dy).numpy(), TOL["bf16"], "dX")
    assert not dX[..., L:].any()
    dW = torch.zeros((B, Co, Ci), dtype=torch.float32, device="cuda")
    hb.conv1x1_bwd(B, Nb, Ci, Co, L, dt, X, strides(Ci), None, dY, strides(Co), None, None, dW, None, ws)
    ref = sum(torch.matmul(dy[n], x[n].transpose(1, 2).contiguous()) for n in range(Nb))
    check(host(dW), ref.numpy(), f32_tol("bf16"), "dW")


@pytest.mark.parametrize("B,Nb,Ci,Co,L,pad", [(2, 5, 12, 20, 4, 4), (1, 3, 4, 36, 12, 0), (3, 7, 64, 132, 132, 4), (2, 3, 136, 4, 1028, 4),
                                              (1, 9, 100, 260, 260, 8), (1, 2, 4, 4, 4, 0), (2, 9, 4, 20, 4, 12), (2, 40, 136, 132, 4, 4)])
def test_forward_and_gradients_of_small_layers(hb, B, Nb, Ci, Co, L, pad):
    """The same for the 128x128 kernel, with four elements in a row of an operand among them: those are read in place, with
    what follows them (NaN here, or past the slice's end) dropped."""
    test_forward_and_gradients(hb, B, Nb, Ci, Co, L, pad)


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(1, 2, 520, 136, 516), (1, 2, 512, 256, 515), (8, 32, 512, 136, 261), (2, 24, 576, 256, 1032)])
def test_wide_data_gradient(hb, B, Nb, Ci, Co, L):
    """More than 128 output channels under at least 512 inputs: products."""
    test_forward_and_gradients(hb, B, Nb, Ci, Co, L, 0)


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(8, 32, 1280, 200, 261), (8, 32, 1280, 192, 261), (8, 32, 1272, 256, 261), (8, 31, 1280, 256, 261),
                                          (4, 64, 1288, 256, 263)])
def test_wide_data_gradient_either_way(hb, B, Nb, Ci, Co, L):
    """Both sides of the rule that streams such gradients (more than 192 channels, 1280 inputs, 768 workgroups, odd rows): with
    its workspace and without, where there is no room for the transposed weights, the same bits."""
    g = torch.Generator(device="cuda")
    g.manual_seed(Ci)
    W = (torch.randn(B, Co, Ci, generator=g, device="cuda") / 16).bfloat16()
    dY = torch.randn(Nb, B, Co, L, generator=g, device="cuda").bfloat16()
    strides = lambda C: (C * L, B * C * L, L, 1)
    n = hb.conv1x1_bwd_workspace_bytes(B, Nb, Ci, Co, L, hb.BF16)
    out = []
    for ws in (torch.empty(max(n, 256), dtype=torch.uint8, device="cuda"), None):
        dX = torch.full((Nb, B, Ci, L), float("nan"), dtype=torch.bfloat16, device="cuda")
        hb.conv1x1_bwd(B, Nb, Ci, Co, L, hb.BF16, None, None, W, dY, strides(Co), dX, strides(Ci), None, None, ws)
        out.append(dX)
    assert torch.equal(*out)
    wt = W[0].float().t().contiguous()
    ref = wt @ dY[0, 0].float()
    assert float((out[0][0, 0].float() - ref).norm() / ref.norm()) <= 2.0 ** -8            # one rounding to bf16


# more than a tile per compute unit, fewer than 256 columns (points, inputs of the data gradient): no room for a tile that ends with the
# matrix, so these stay on the register-staged kernel
@pytest.mark.parametrize("B,Nb,Ci,Co,L,pad", [(1, 260, 256, 256, 252, 4), (2, 131, 264, 256, 196, 0), (1, 260, 252, 256, 260, 0)])
def test_fewer_columns_than_a_tile(hb, B, Nb, Ci, Co, L, pad):
    test_forward_and_gradients(hb, B, Nb, Ci, Co, L, pad)


@pytest.mark.parametrize("B,M,Fx,Fy", [(9, 7424, 256, 252), (3, 22300, 256, 196)])
def test_linear_of_fewer_columns_than_a_tile(hb, B, M, Fx, Fy):
    """The same with a bias per column."""
    gen = torch.Generator(device="cuda").manual_seed(8)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()
    x, w, bias = r(B, M, Fx), r(B, Fx, Fy) / 16, r(B, Fy)
    y = torch.full((B, M, Fy), float("nan"), dtype=torch.bfloat16, device="cuda")
    hb.linear_fwd(B, M, Fx, Fy, DT["bf16"], x, w, bias, y, hb.ACT_RELU)
    for b in range(B):
        ref = x[b].double() @ w[b].double() + bias[b].double()
        mag = x[b].double().abs() @ w[b].double().abs() + bias[b].double().abs()
        # a rounding to bf16 of an fp32 sum of Fx + 1 terms
        assert ((y[b].double() - ref.clamp_min(0)).abs() <= 2.0 ** -8 * ref.abs() + (Fx + 1) * 2.0 ** -24 * mag).all()
