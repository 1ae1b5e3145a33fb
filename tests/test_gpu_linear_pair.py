"""Both gradients of a Linear in one launch: the bits of the two launches, at tile edges and remainders."""
import pytest
import torch

from paper_2102_02344_amd import binding as hb

DEV = "cuda"


def _same(a, b, what):
    kind = torch.int32 if a.dtype == torch.float32 else torch.int16
    assert torch.equal(a.view(kind), b.view(kind)), what


# 64- and 128-row tiles of either gradient, partial tiles along every dimension, one k-tile, a workgroup count that is no multiple of 8
SHAPES = [(1, 64, 8, 8), (1, 65, 72, 200), (3, 127, 256, 72), (5, 693, 384, 1536), (4, 3000, 256, 1024), (8, 2048, 256, 1024), (2, 1000, 1032, 264),
          (8, 1024, 1024, 256)]


@pytest.mark.gpu
@pytest.mark.parametrize("B,M,Fx,Fy", SHAPES)
def test_one_launch(B, M, Fx, Fy):
    assert hb.linear_bwd_pair_supported(B, M, Fx, Fy, hb.BF16)
    g = torch.Generator(device=DEV).manual_seed(M + Fx)
    r = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
    x, w, dy = r(B, M, Fx), r(B, Fx, Fy), r(B, M, Fy)
    ws = torch.empty(max(4, hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.BF16)), dtype=torch.uint8, device=DEV)

    def both(separate, db=True):
        dx = torch.full((B, M, Fx), float("nan"), dtype=torch.bfloat16, device=DEV)
        dw, dbias = torch.full((B, Fx, Fy), float("nan"), device=DEV), torch.zeros(B, Fy, device=DEV)
        if separate:
            hb.linear_bwd(B, M, Fx, Fy, hb.BF16, None, w, dy, dx, None, None, None)
            hb.linear_bwd(B, M, Fx, Fy, hb.BF16, x, None, dy, None, dw, dbias if db else None, ws)
        else:
            hb.linear_bwd(B, M, Fx, Fy, hb.BF16, x, w, dy, dx, dw, dbias if db else None, ws)
        return dx, dw, dbias

    for db in (True, False):
        for a, b, what in zip(both(True, db), both(False, db), ("dX", "dW", "dbias")):
            _same(a, b, (what, db))


@pytest.mark.gpu
@pytest.mark.parametrize("off", ["x", "w", "dy", "dx", "dw"])
def test_other_alignments(off):
    """Operands that start off 16 bytes take two launches, results that do take narrower stores; the values do not change."""
    B, M, Fx, Fy = 2, 200, 64, 136
    g = torch.Generator(device=DEV).manual_seed(1)

    def at(name, dtype, *s):
        n = 1
        for v in s:
            n *= v
        buf = torch.randn(n + 8, generator=g, device=DEV).to(dtype)
        return (buf[4 if dtype == torch.bfloat16 else 2:][:n] if name == off else buf[:n]).view(*s)
    x, w, dy = at("x", torch.bfloat16, B, M, Fx), at("w", torch.bfloat16, B, Fx, Fy), at("dy", torch.bfloat16, B, M, Fy)
    dx, dw = at("dx", torch.bfloat16, B, M, Fx), at("dw", torch.float32, B, Fx, Fy)
    ws = torch.empty(max(4, hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.BF16)), dtype=torch.uint8, device=DEV)
    hb.linear_bwd(B, M, Fx, Fy, hb.BF16, x, w, dy, dx, dw, None, ws)
    dx2, dw2 = torch.empty_like(dx), torch.empty_like(dw)
    hb.linear_bwd(B, M, Fx, Fy, hb.BF16, x.clone(), w.clone(), dy.clone(), dx2, dw2, None, ws)
    _same(dx.contiguous(), dx2, "dX")
    _same(dw.contiguous(), dw2, "dW")


def test_which_products():
    ok = lambda *a: hb.linear_bwd_pair_supported(*a)
    assert ok(8, 2048, 256, 1024, hb.BF16) and ok(1, 64, 8, 8, hb.BF16)
    assert not ok(8, 2048, 256, 1024, hb.F32) and not ok(1, 63, 256, 256, hb.BF16) and not ok(1, 64, 12, 8, hb.BF16)
    assert not ok(8, 2048, 1024, 256, hb.BF16)          # 2304 tiles
    assert not ok(16, 4096, 512, 2048, hb.BF16) and not ok(1, 8193, 64, 64, hb.BF16) and not ok(0, 64, 8, 8, hb.BF16)


def test_split_weight_gradients_are_no_pair():
    """What is announced as one launch is one: a weight gradient of more than 320 tiles of 128 x 128 keeps its split over the rows."""
    assert not hb.linear_bwd_pair_supported(9, 504, 384, 1536, hb.BF16) and not hb.linear_bwd_pair_supported(7, 808, 512, 2048, hb.BF16)
    split = 0
    for E in (256, 384, 512):
        for B in range(1, 17):
            for M in range(128, 4097, 56):
                for Fx, Fy in ((E, 4 * E), (4 * E, E)):
                    if hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.BF16) and B * -(-Fx // 128) * -(-Fy // 128) > 320:
                        split += 1
                        assert not hb.linear_bwd_pair_supported(B, M, Fx, Fy, hb.BF16), (B, M, Fx, Fy)
    assert split > 100


@pytest.mark.gpu
def test_where_the_weight_gradient_is_split():
    B, M, Fx, Fy = 9, 504, 384, 1536
    g = torch.Generator(device=DEV).manual_seed(9)
    r = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
    x, w, dy = r(B, M, Fx), r(B, Fx, Fy), r(B, M, Fy)
    ws = torch.empty(hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.BF16), dtype=torch.uint8, device=DEV)
    dx, dx2, dw, dw2 = torch.empty_like(x), torch.empty_like(x), torch.empty(B, Fx, Fy, device=DEV), torch.empty(B, Fx, Fy, device=DEV)
    hb.linear_bwd(B, M, Fx, Fy, hb.BF16, x, w, dy, dx, dw, None, ws)
    hb.linear_bwd(B, M, Fx, Fy, hb.BF16, None, w, dy, dx2, None, None, None)
    hb.linear_bwd(B, M, Fx, Fy, hb.BF16, x, None, dy, None, dw2, None, ws)
    _same(dx, dx2, "dX")
    _same(dw, dw2, "dW")


def test_one_round_of_large_tiles_each():
    """Widths that are no whole tiles of 128, both products a round of 128 x 128 tiles, 40 k-tiles together: two launches."""
    ok = lambda *a: hb.linear_bwd_pair_supported(*a, hb.BF16)
    assert not ok(9, 2138, 104, 2912) and not ok(5, 2433, 232, 1944) and not ok(15, 1445, 128, 1856)
    assert ok(6, 1536, 384, 1536) and ok(3, 2431, 512, 1536)            # whole tiles
    assert ok(13, 811, 232, 912)                                       # 28 k-tiles
    assert ok(14, 1693, 88, 2440) and ok(8, 2138, 56, 2912)             # more than a round of one, smaller tiles for the other
