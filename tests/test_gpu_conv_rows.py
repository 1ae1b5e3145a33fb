"""Forward and weight gradient of the 4x4 / stride 2 convolution from image rows, at the image shapes the row kernels lay
out differently: rows of one to 32 sixteen-byte pieces, samples smaller and larger than a tile of columns or of pixels
(one-row samples among them), odd image heights, channels and samples that fill neither tile, reductions split and not.
Same reference and tolerance as the operator's other sizes; the split reduction also against the unsplit one."""
import numpy as np
import pytest
import torch

import hfta_inputs as hi
import test_gpu_ops as ops
from oracle import array as oa
from util import DT, TOL, check, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


@pytest.mark.parametrize("B,Nb,Ci,Co,H,W", [
    (2, 5, 7, 33, 8, 8), (1, 9, 6, 70, 16, 8), (1, 3, 5, 40, 64, 8), (2, 7, 9, 130, 4, 16), (1, 5, 13, 65, 17, 16),
    (1, 9, 6, 34, 2, 32), (2, 3, 11, 36, 4, 32), (1, 3, 3, 66, 32, 32), (1, 5, 10, 33, 2, 64), (1, 2, 9, 48, 65, 64),
    (1, 3, 5, 32, 2, 128), (1, 1, 6, 33, 2, 256), (1, 2, 130, 34, 8, 8), (1, 34, 130, 40, 8, 16)])
def test_forward_and_weight_gradient(hb, B, Nb, Ci, Co, H, W):
    print(f"conv rows B={B} Nb={Nb} Ci={Ci} Co={Co} H={H} W={W}", flush=True)
    x = hi.normal(131, (Nb, B * Ci, H, W), "bf16")
    w = hi.normal(132, (B * Co, Ci, 4, 4), "bf16", 1.0 / np.sqrt(Ci * 16))
    b = hi.normal(133, (B * Co,), "bf16")
    ry = oa.conv2d_fwd(B, x, w, b, 2, 1)
    dy = hi.normal(134, ry.shape, "bf16")
    X, Wt, Bi, dY = dev(x, "bf16"), dev(w, "bf16"), dev(b, "bf16"), dev(dy, "bf16")
    args = (B, Nb, Ci, Co, H, W, 4, 4, 2, 1, DT["bf16"])
    wsf, wsb = ops.conv_workspaces(hb, "lowered", args)
    Y, Ys = ops.empty(ry.shape, "bf16"), ops.empty(ry.shape, "bf16")
    hb.conv2d_grouped_fwd(*args, X, Wt, Bi, Y)
    check(host(Y), ry, TOL["bf16"], "Y")
    hb.conv2d_grouped_fwd(*args, X, Wt, Bi, Ys, workspace=wsf)       # long reductions: split over k
    check(host(Ys), ry, TOL["bf16"], "Y split")
    dW = ops.empty(w.shape, torch.float32)
    hb.conv2d_grouped_bwd(*args, X, Wt, dY, None, dW, None, wsb)
    check(host(dW), oa.conv2d_bwd(B, x, w, dy, 2, 1)[1], ops.f32_tol("bf16"), "dW")
