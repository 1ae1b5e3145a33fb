"""Data gradient of the 4x4 / stride 2 convolution at the image sizes its plane kernel treats differently (rows of
one, two and eight 16-byte pieces, four-pixel rows in whole images, images smaller and larger than a tile), at
ragged samples and channels, and below and above one workgroup per compute unit.  Same reference and tolerance
as the operator's other sizes."""
import pytest

import test_gpu_ops as ops

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


@pytest.mark.parametrize("B,Nb,Ci,Co,H", [
    (1, 1, 32, 2, 8), (2, 5, 40, 50, 8), (2, 7, 130, 34, 8), (1, 3, 72, 18, 16), (1, 2, 33, 66, 32), (1, 1, 32, 20, 64),
    (1, 1, 96, 16, 128), (5, 30, 260, 36, 8)])
def test_data_gradient(hb, B, Nb, Ci, Co, H):
    ops.test_conv2d_grouped(hb, "bf16", B, Nb, Ci, Co, H, 4, 2, 1, "implicit")
