"""Attention core at the head and sequence sizes where the one-kernel form changes path: one token, whole and
partial 16-token blocks, past each register size (64, 128, 256 tokens), heads of one 16-byte piece up to 64
columns, and the sizes it leaves to the batched products (257 tokens, 12 or 72 columns).  Same oracle and
tolerance as the operator's other sizes (the kernel rounds where the oracle does)."""
import pytest
import torch

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


@pytest.mark.parametrize("causal", [0, 1])
def test_probabilities_far_below_the_maximum(hb, causal):
    """Every probability is the bf16 rounding of a value within e of exp(s - max) / sum.  Whole-number queries and keys
    and 16 columns (a scale of 1/4) make the scores and their differences exact, so that what is left is rounding of the
    softmax itself: one unit (2^-23) of the exponential above and below the line, six additions below it, the
    reciprocal and the product, half a unit each: e = (2 + 2 + 6 + 2) 2^-24.  An exponential whose error grows with its
    argument fails here: at exp(-60) the argument's own rounding in base 2 is 2.6e-6."""
    B, N, S, E, H = 2, 32, 16, 128, 8
    g = torch.Generator().manual_seed(11)
    qkv = torch.randint(-8, 9, (B, N, S, 3 * E), generator=g).float()
    P = torch.full((B, N, H, S, S), float("nan"), dtype=torch.bfloat16, device="cuda")
    ctx = torch.empty(B, N, S, E, dtype=torch.bfloat16, device="cuda")
    hb.attention_fwd(B, N, S, E, H, 1, qkv.to(torch.bfloat16).cuda(), P, ctx, causal)
    q, k = (t.reshape(B, N, S, H, E // H).permute(0, 1, 3, 2, 4).double() for t in qkv.split(E, -1)[:2])
    s = (q @ k.transpose(-1, -2)).bfloat16().double() / 4        # stored scores are bf16
    if causal:
        s = s.masked_fill(~torch.ones(S, S, dtype=torch.bool).tril(), float("-inf"))
    p = torch.softmax(s, -1)
    e = 12 * 2.0 ** -24
    lo, hi = (torch.from_numpy((p * f).numpy()).to(torch.bfloat16) for f in (1 - e, 1 + e))
    got = P.cpu()
    seen = p > 1e-30                                             # below: bf16 and fp32 near their smallest normal numbers
    assert int((seen & (p < 1e-12)).sum()) > 10000
    assert bool(((got >= lo) & (got <= hi))[seen].all())
    assert bool((got[p == 0] == 0).all())


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("S", [20, 70, 200])
@pytest.mark.parametrize("what", ["query nan", "query inf", "key nan", "key inf"])
def test_values_that_are_not_finite(hb, what, S, causal):
    """A NaN or an infinity in one query or key reaches the probabilities that the batched products give it (which the
    same call takes with its output 8 bytes off): the row's own, none behind the causal mask, and no other row's."""
    B, N, E, H, at = 1, 2, 48, 2, S // 2 + 3
    g = torch.Generator().manual_seed(13)
    qkv = torch.randn(B, N, S, 3 * E, generator=g).bfloat16()
    qkv[0, 1, at, (0 if what.startswith("query") else E) + 5] = float(what.split()[1])
    qkv = qkv.cuda()
    P = [torch.full((B, N, H, S, S), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    for p, off in zip(P, (0, 4)):
        ctx = torch.empty(B * N * S * E + 8, dtype=torch.bfloat16, device="cuda")[off:]
        hb.attention_fwd(B, N, S, E, H, 1, qkv, p, ctx, causal)
    a, b = (p.cpu().float() for p in P)
    assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a == 0, b == 0)
    assert bool(a.isnan().any()) and not bool(a[:, 0].isnan().any())
    ok = ~a.isnan()
    assert bool(((a - b).abs() <= 2.0 ** -7 * b.abs())[ok].all())
