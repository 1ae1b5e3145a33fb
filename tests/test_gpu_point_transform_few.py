"""Point transforms of few input channels (the coordinates): rows of whole and of partial four-point pieces, more outputs than
a workgroup takes, several workgroups a row, and rows too short for the kernel.  Same reference and tolerance as the others."""
import pytest

import test_gpu_ops as ops

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


@pytest.mark.parametrize("B,Nb,Ci,Co,L", [(2, 3, 3, 3, 2500), (3, 2, 3, 3, 1023), (1, 5, 4, 17, 7), (2, 2, 1, 33, 4), (1, 2, 3, 5, 3), (1, 1, 2, 2, 1026)])
def test_few_channels(hb, B, Nb, Ci, Co, L):
    ops.test_point_transform(hb, "bf16", B, Nb, Ci, Co, L)
