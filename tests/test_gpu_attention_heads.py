"""Attention core at the head and sequence sizes where the one-kernel form changes path: one token, whole and
partial 16-token blocks, past each register size (64, 128, 256 tokens), heads of one 16-byte piece up to 64
columns, and the sizes it leaves to the batched products (257 tokens, 12 or 72 columns).  Same oracle and
tolerance as the operator's other sizes (the kernel rounds where the oracle does)."""
import pytest

import test_gpu_transformer as tr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


@pytest.mark.parametrize("B,N,S,E,H,causal", [
    (1, 2, 1, 64, 1, 1), (2, 1, 16, 64, 1, 1), (2, 2, 17, 128, 2, 0), (1, 2, 65, 80, 2, 1), (1, 3, 128, 16, 2, 0),
    (1, 2, 129, 128, 2, 1), (2, 2, 250, 256, 4, 1), (1, 1, 256, 64, 1, 0), (1, 1, 257, 64, 1, 1), (1, 2, 40, 24, 2, 1),
    (1, 2, 33, 144, 2, 1)])
def test_attention_sizes(hb, B, N, S, E, H, causal):
    tr.test_attention_core(hb, "bf16", B, N, S, E, H, causal)
