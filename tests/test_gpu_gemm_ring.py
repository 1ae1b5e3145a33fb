"""The 256x256 products on a ring of LDS slots, at the sizes where the ring, the tile walk and the epilogue can go wrong: a second
round of workgroups, one column past a tile, k that ends inside a k-tile, the shortest reduction, split reductions, output
rows of 8-byte alignment, batches that do not divide among the XCDs."""
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


@pytest.mark.parametrize("B,M,Fx,Fy,relu", [(50, 300, 264, 520, True), (65, 257, 256, 776, False), (200, 448, 520, 192, False),
                                            (97, 320, 260, 256, False), (33, 768, 256, 520, True), (4, 4104, 512, 264, False)])
def test_linear(hb, B, M, Fx, Fy, relu):
    print(f"ring products B={B} M={M} Fx={Fx} Fy={Fy}", flush=True)
    gen = torch.Generator().manual_seed(11)
    dt = DT["bf16"]
    r = lambda *s: torch.randn(s, generator=gen).bfloat16()
    X, W, b, dY = r(B, M, Fx), (r(B, Fx, Fy).float() / np.sqrt(Fx)).bfloat16(), r(B, Fy), r(B, M, Fy)
    Xd, Wd, bd, dYd = X.cuda(), W.cuda(), b.cuda(), dY.cuda()
    x, w, dy = X.double(), W.double(), dY.double()
    ws = torch.empty(max(hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, dt), 4), dtype=torch.uint8, device="cuda")
    Y = torch.full((B, M, Fy), float("nan"), dtype=torch.bfloat16, device="cuda")
    hb.linear_fwd(B, M, Fx, Fy, dt, Xd, Wd, bd, Y, act=hb.ACT_RELU if relu else hb.ACT_NONE)
    y = torch.matmul(x, w) + b.double()[:, None, :]
    check(host(Y), (y.clamp(min=0) if relu else y).numpy(), TOL["bf16"], "Y")
    dX = torch.full((B, M, Fx), float("nan"), dtype=torch.bfloat16, device="cuda")
    hb.linear_bwd(B, M, Fx, Fy, dt, None, Wd, dYd, dX, None, None, ws)
    check(host(dX), torch.matmul(dy, w.transpose(1, 2).contiguous()).numpy(), TOL["bf16"], "dX")
    dW = torch.full((B, Fx, Fy), float("nan"), device="cuda")
    hb.linear_bwd(B, M, Fx, Fy, dt, Xd, None, dYd, None, dW, None, ws)
    check(host(dW), torch.matmul(x.transpose(1, 2).contiguous(), dy).numpy(), f32_tol("bf16"), "dW")


@pytest.mark.parametrize("B,M,Fx,Fy,relu,shift", [(8, 2048, 256, 1024, True, 0), (16, 768, 512, 1024, False, 0), (12, 1024, 384, 1016, False, 0),
                                                  (4, 2048, 256, 2044, True, 0), (7, 2000, 256, 1016, True, 4), (13, 1024, 264, 1024, False, 4)])
def test_bias_after_the_sum(hb, B, M, Fx, Fy, relu, shift):
    """One output tile per workgroup (192 to 256 tiles): the bias is added to the finished sum.  The partial sums pass through
    2^27, where a bias of a few units added at the start would be rounded away, and return to zero: the output is the bias.
    `shift`: elements by which the output starts off 16 bytes."""
    print(f"bias after the sum B={B} M={M} Fx={Fx} Fy={Fy} shift={shift}", flush=True)
    assert 192 <= B * ((M + 255) // 256) * ((Fy + 255) // 256) <= torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator().manual_seed(7)
    X = torch.full((B, M, Fx), 1024.0, dtype=torch.bfloat16)
    W = torch.full((B, Fx, Fy), 1024.0, dtype=torch.bfloat16)
    W[:, Fx // 2:] = -1024.0
    b = torch.randint(1, 5, (B, Fy), generator=gen).bfloat16()
    Y = torch.full((B * M * Fy + shift,), float("nan"), dtype=torch.bfloat16, device="cuda")[shift:].view(B, M, Fy)
    hb.linear_fwd(B, M, Fx, Fy, DT["bf16"], X.cuda(), W.cuda(), b.cuda(), Y, act=hb.ACT_RELU if relu else hb.ACT_NONE)
    assert torch.equal(Y.cpu(), b[:, None, :].expand(B, M, Fy))


@pytest.mark.parametrize("B,M,Fx,Fy", [(64, 300, 256, 1024), (65, 300, 256, 1024), (33, 520, 512, 1000)])
def test_weight_and_bias_gradient(hb, B, M, Fx, Fy):
    """Column sums of dY beside the weight gradient, on both sides of one tile per workgroup: the same dW bits without them."""
    print(f"weight and bias gradient B={B} M={M} Fx={Fx} Fy={Fy}", flush=True)
    gen = torch.Generator().manual_seed(3)
    X, dY = torch.randn(B, M, Fx, generator=gen).bfloat16().cuda(), torch.randn(B, M, Fy, generator=gen).bfloat16().cuda()
    ws = torch.empty(max(hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, DT["bf16"]), 4), dtype=torch.uint8, device="cuda")
    dW, dW2 = (torch.full((B, Fx, Fy), float("nan"), device="cuda") for _ in range(2))
    db = torch.full((B, Fy), float("nan"), device="cuda")
    hb.linear_bwd(B, M, Fx, Fy, DT["bf16"], X, None, dY, None, dW, db, ws)
    hb.linear_bwd(B, M, Fx, Fy, DT["bf16"], X, None, dY, None, dW2, None, ws)
    assert torch.equal(dW, dW2)
    x, dy = X.cpu().double(), dY.cpu().double()
    check(host(dW), torch.matmul(x.transpose(1, 2).contiguous(), dy).numpy(), f32_tol("bf16"), "dW")
    check(host(db), dy.sum(1).numpy(), f32_tol("bf16"), "db")
