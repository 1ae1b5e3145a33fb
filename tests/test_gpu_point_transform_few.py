"""Point transforms of few input channels (the coordinates): rows of whole and of partial four-point pieces, more outputs than
a workgroup takes, several workgroups a row, and rows too short for the kernel.  Same reference and tolerance as the others."""
import pytest
import torch

import test_gpu_ops as ops

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(2, 3, 3, 3, 2500), (3, 2, 3, 3, 1023), (1, 5, 4, 17, 7), (2, 2, 1, 33, 4), (1, 2, 3, 5, 3), (1, 1, 2, 2, 1026)])
def test_few_channels(hb, B, Nb, Ci, Co, L):
    ops.test_point_transform(hb, "bf16", B, Nb, Ci, Co, L)


@pytest.mark.parametrize("B,Nb,L", [(4, 16, 2499), (2, 24, 1023), (3, 16, 1026)])
def test_rows_of_partial_pieces_round_as_the_product(hb, B, Nb, L):
    """Bit for bit the k=1 convolution of the same weights, whose single form keeps the matrix kernels on such rows.  The first
    and third products cancel and the second lies at their last bits in fp32, so that every rounding of the sum shows."""
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    X = torch.randn(Nb, B, 3, L, generator=g, device="cuda")
    X[:, :, 1] *= 2.0 ** -14
    X[:, :, 2] = X[:, :, 0]
    T = torch.randn(B, Nb, 3, 3, generator=g, device="cuda")
    T[..., 2] = -T[..., 0]
    X, T = X.bfloat16(), T.bfloat16()
    cs = (3 * L, B * 3 * L, L, 1)
    Y, ref = torch.empty_like(X), torch.empty_like(X)
    hb.point_transform_fwd(B, Nb, 3, 3, L, hb.BF16, X, cs, T, Y, cs)
    for n in range(Nb):
        hb.conv1x1_fwd(B, 1, 3, 3, L, hb.BF16, X[n], cs, T[:, n].contiguous(), None, ref[n], cs)
    assert torch.equal(Y.view(torch.int16), ref.view(torch.int16))
