"""4x4 / stride 2 convolutions and their data gradients in row tiles of 64 (few tiles) and of 128 (many): against float64, and the
same bits whichever the launch takes."""
import pytest
import torch
import torch.nn.functional as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


# rows of 128 + 2, of 64 + 2, a multiple of both, fewer than a tile of 128; images of 4x4, 8x8, 16x16 outputs; many: 256 tiles and more
@pytest.mark.parametrize("Nb,Ci,Co,H,many", [(5, 66, 130, 16, 72), (9, 120, 66, 8, 200), (2, 100, 128, 32, 64), (17, 72, 96, 8, 66)])
def test_row_tiles(hb, Nb, Ci, Co, H, many):
    print(f"conv {Nb} x {Ci} -> {Co} at {H}", flush=True)
    gen = torch.Generator().manual_seed(11)
    r = lambda *s: torch.randn(s, generator=gen).bfloat16()
    x, w, dy = r(Nb, Ci, H, H), 0.05 * r(Co, Ci, 4, 4), r(Nb, Co, H // 2, H // 2)
    got = []
    for B in (1, many):
        X, W, dY = (v.repeat(*n).contiguous().cuda() for v, n in ((x, (1, B, 1, 1)), (w, (B, 1, 1, 1)), (dy, (1, B, 1, 1))))
        Y, dX = torch.full_like(dY, float("nan")), torch.full_like(X, float("nan"))
        dims = (B, Nb, Ci, Co, H, H, 4, 4, 2, 1, 1)
        need = max(hb.conv2d_grouped_fwd_workspace_bytes(*dims), hb.conv2d_grouped_bwd_min_workspace_bytes(*dims), 4)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        hb.conv2d_grouped_fwd(*dims, X, W, None, Y, workspace=ws)
        hb.conv2d_grouped_bwd(*dims, None, W, dY, dX, None, None, workspace=ws)
        got.append((Y.cpu().view(Nb, B, Co, H // 2, H // 2), dX.cpu().view(Nb, B, Ci, H, H)))
    x, w, dy = x.double(), w.double(), dy.double()
    for few, lot, f, a in ((got[0][0], got[1][0], F.conv2d, x), (got[0][1], got[1][1], F.conv_transpose2d, dy)):
        ref, mag = f(a, w, stride=2, padding=1), f(a.abs(), w.abs(), stride=2, padding=1)
        # the result rounded to eight bits (half a unit: 2^-8 of 1.0 whose unit is 2^-7), sums of at most 16 Ci (4 Co) products in fp32 (2^-24 each)
        assert ((few[:, 0].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 16 * max(Ci, Co) * 2.0 ** -24 * mag).all()
        for b in range(lot.shape[1]):
            assert torch.equal(few[:, 0].contiguous().view(torch.int16), lot[:, b].contiguous().view(torch.int16)), b


# images of whole tiles of 16 rows, of one row more, of less than one; rows of more than a tile; channels of the last stage: 4, 8 of 8
@pytest.mark.parametrize("Nb,Ci,Co,H,W,many", [(20, 3, 20, 64, 64, 13), (8, 1, 8, 34, 36, 32), (9, 4, 12, 18, 68, 29), (16, 2, 24, 14, 4, 32)])
def test_few_channels_rows(hb, Nb, Ci, Co, H, W, many):
    """Data gradient of a convolution of at most four channels, one and two rows of pixels a thread: as above."""
    print(f"conv {Nb} x {Ci} -> {Co} at {H} x {W}", flush=True)
    gen = torch.Generator().manual_seed(12)
    r = lambda *s: torch.randn(s, generator=gen).bfloat16()
    w, dy = 0.05 * r(Co, Ci, 4, 4), r(Nb, Co, H // 2, W // 2)
    got = []
    for B in (1, many):
        Wt, dY = w.repeat(B, 1, 1, 1).cuda(), dy.repeat(1, B, 1, 1).cuda()
        dX = torch.full((Nb, B * Ci, H, W), float("nan"), dtype=torch.bfloat16, device="cuda")
        dims = (B, Nb, Ci, Co, H, W, 4, 4, 2, 1, 1)
        ws = torch.empty(max(hb.conv2d_grouped_bwd_min_workspace_bytes(*dims), 4), dtype=torch.uint8, device="cuda")
        hb.conv2d_grouped_bwd(*dims, None, Wt, dY, dX, None, None, workspace=ws)
        got.append(dX.cpu().view(Nb, B, Ci, H, W))
    w, dy = w.double(), dy.double()
    ref, mag = F.conv_transpose2d(dy, w, stride=2, padding=1), F.conv_transpose2d(dy.abs(), w.abs(), stride=2, padding=1)
    assert ((got[0][:, 0].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 4 * Co * 2.0 ** -24 * mag).all()
    for b in range(many):
        assert torch.equal(got[0][:, 0].contiguous().view(torch.int16), got[1][:, b].contiguous().view(torch.int16)), b


# four splits of 128 k-tiles, two of 68; channels of two row tiles of 128 and three of 64, and of one and two; `many`: 256 workgroups and more,
# of as many splits
@pytest.mark.parametrize("Nb,Ci,Co,H,many", [(9, 256, 130, 8, 20), (5, 136, 130, 16, 40), (17, 264, 100, 8, 30)])
def test_row_tiles_of_a_split_reduction(hb, Nb, Ci, Co, H, many):
    """The forward's 64-row tiles with the reduction split over workgroups: the same bits as 128-row tiles of that split, and float64."""
    print(f"conv {Nb} x {Ci} -> {Co} at {H}, split", flush=True)
    gen = torch.Generator().manual_seed(13)
    r = lambda *s: torch.randn(s, generator=gen).bfloat16()
    x, w, bias = r(Nb, Ci, H, H), 0.05 * r(Co, Ci, 4, 4), r(Co)
    got = []
    for B in (1, many):
        X, W, bi = x.repeat(1, B, 1, 1).cuda(), w.repeat(B, 1, 1, 1).cuda(), bias.repeat(B).cuda()
        dims = (B, Nb, Ci, Co, H, H, 4, 4, 2, 1, 1)
        ws = torch.full((hb.conv2d_grouped_fwd_workspace_bytes(*dims),), 255, dtype=torch.uint8, device="cuda")
        for work in (ws, None):
            Y = torch.full((Nb, B * Co, H // 2, H // 2), float("nan"), dtype=torch.bfloat16, device="cuda")
            hb.conv2d_grouped_fwd(*dims, X, W, bi, Y, 1, workspace=work)
            got.append(Y.cpu().view(Nb, B, Co, H // 2, H // 2))
    assert not torch.equal(got[0], got[1]) and not torch.equal(got[2], got[3])      # the split is another order of the sums
    xd, wd, bd = x.double(), w.double(), bias.double()
    ref = F.conv2d(xd, wd, bd, stride=2, padding=1)
    mag = F.conv2d(xd.abs(), wd.abs(), bd.abs(), stride=2, padding=1)
    for few in got[:2]:
        assert ((few[:, 0].double() - ref.clamp_min(0)).abs() <= 2.0 ** -8 * ref.abs() + 16 * Ci * 2.0 ** -24 * mag).all()
    for few, lot in ((got[0], got[2]), (got[1], got[3])):
        for b in range(many):
            assert torch.equal(few[:, 0].contiguous().view(torch.int16), lot[:, b].contiguous().view(torch.int16)), b
