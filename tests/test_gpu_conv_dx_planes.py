"""Data gradient of the 4x4 / stride 2 convolution at the image sizes its plane kernel treats differently (rows of
one, two and eight 16-byte pieces, four-pixel rows in whole images, images smaller and larger than a tile), at
ragged samples and channels, below one workgroup per compute unit (two k-tiles of weights in registers) and above
(one), with tiles of 64 and of 128 rows; and of four-pixel rows in images taller than a tile, which the gathering
kernel keeps.  Same reference and tolerance as the operator's other sizes."""
import numpy as np
import pytest
import torch

import hfta_inputs as hi
import test_gpu_ops as ops
from oracle import array as oa
from util import TOL, check, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


@pytest.mark.parametrize("B,Nb,Ci,Co,H", [
    (1, 1, 32, 2, 8), (2, 5, 40, 50, 8), (2, 7, 130, 34, 8), (1, 3, 72, 18, 16), (1, 2, 33, 66, 32), (1, 1, 32, 20, 64),
    (1, 1, 96, 16, 128), (5, 30, 260, 36, 8),
    # workgroups: rows / 128 (or 64) x samples' pixels / 64 x 2 x models = 288, 288, 260, 270
    (6, 30, 260, 36, 8), (16, 33, 40, 18, 8), (5, 13, 130, 34, 16), (9, 15, 50, 20, 16)])
def test_data_gradient(hb, B, Nb, Ci, Co, H):
    ops.test_conv2d_grouped(hb, "bf16", B, Nb, Ci, Co, H, 4, 2, 1, "implicit")


@pytest.mark.parametrize("B,Nb,Ci,Co", [(2, 3, 40, 18), (1, 2, 130, 6)])
def test_data_gradient_of_tall_images(hb, B, Nb, Ci, Co):
    H, W = 64, 8
    x = hi.normal(101, (Nb, B * Ci, H, W), "bf16")
    w = hi.normal(102, (B * Co, Ci, 4, 4), "bf16", 1.0 / np.sqrt(Ci * 16))
    dy = hi.normal(104, (Nb, B * Co, H // 2, W // 2), "bf16")
    dX = ops.empty(x.shape, "bf16")
    _, ws = ops.conv_workspaces(hb, "implicit", (B, Nb, Ci, Co, H, W, 4, 4, 2, 1, 1))
    hb.conv2d_grouped_bwd(B, Nb, Ci, Co, H, W, 4, 4, 2, 1, 1, dev(x, "bf16"), dev(w, "bf16"), dev(dy, "bf16"), dX, None, None, ws)
    check(host(dX), oa.conv2d_bwd(B, x, w, dy, 2, 1)[0], TOL["bf16"], "dX")


@pytest.mark.parametrize("B,Nb,Ci,Co,H,W,shift", [
    (2, 3, 3, 64, 64, 64, 0), (1, 2, 1, 5, 6, 10, 0), (2, 2, 4, 33, 18, 70, 0), (1, 3, 2, 16, 34, 2, 0), (2, 1, 3, 17, 20, 132, 0),
    (1, 2, 3, 16, 64, 68, 1)])
def test_data_gradient_of_few_channels(hb, B, Nb, Ci, Co, H, W, shift):
    """Up to four input channels: output channels short of a stage, rows of one, an odd and an even number of gradient columns,
    tiles that end past the image, and a gradient that starts off four bytes."""
    x = hi.normal(111, (Nb, B * Ci, H, W), "bf16")
    w = hi.normal(112, (B * Co, Ci, 4, 4), "bf16", 1.0 / np.sqrt(Ci * 16))
    dy = hi.normal(114, (Nb, B * Co, H // 2, W // 2), "bf16")
    dX = ops.empty(x.shape, "bf16")
    _, ws = ops.conv_workspaces(hb, "implicit", (B, Nb, Ci, Co, H, W, 4, 4, 2, 1, 1))
    flat = dev(dy, "bf16").reshape(-1)
    dY = flat.new_empty(flat.numel() + shift)[shift:]
    dY.copy_(flat)
    hb.conv2d_grouped_bwd(B, Nb, Ci, Co, H, W, 4, 4, 2, 1, 1, dev(x, "bf16"), dev(w, "bf16"), dY.view(dy.shape), dX, None, None, ws)
    check(host(dX), oa.conv2d_bwd(B, x, w, dy, 2, 1)[0], TOL["bf16"], "dX")


def test_data_gradient_of_few_channels_of_a_large_image(hb):
    """One sample whose gradient is 2 GiB: the last rows are, bit for bit, those of an image that has only these."""
    Ci, Co, H, q = 3, 64, 8192, 34
    print("few channels, 2 GiB of gradient", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(2)
    dY = torch.randn((Co, H // 2, H // 2), generator=gen, device="cuda", dtype=torch.bfloat16)
    W = torch.randn((Co, Ci, 4, 4), generator=gen, device="cuda", dtype=torch.bfloat16)
    dX = torch.full((Ci, H, H), float("nan"), device="cuda", dtype=torch.bfloat16)
    hb.conv2d_grouped_bwd(1, 1, Ci, Co, H, H, 4, 4, 2, 1, 1, dX, W, dY, dX, None, None, None)
    rows = dY[:, -q:].contiguous()
    part = torch.full((Ci, 2 * q, H), float("nan"), device="cuda", dtype=torch.bfloat16)
    hb.conv2d_grouped_bwd(1, 1, Ci, Co, 2 * q, H, 4, 4, 2, 1, 1, part, W, rows, part, None, None, None)
    assert torch.equal(dX[:, 2 - 2 * q:], part[:, 2:])
    x = torch.nn.functional.conv_transpose2d(rows[:, -4:, -4:].float().cpu()[None], W.float().cpu(), stride=2, padding=1)[0]
    check(host(dX[:, -6:, -6:]), x[:, 2:, 2:].double().numpy(), TOL["bf16"], "corner")
