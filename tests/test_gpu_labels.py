"""Cross-entropy with a label that is no class: its model's loss is NaN, its gradient is that of no class, the other models and
rows do not notice."""
import pytest
import torch

from paper_2102_02344_amd import binding as hb

pytestmark = pytest.mark.gpu
DEV = "cuda"
TDT = {hb.F32: torch.float32, hb.BF16: torch.bfloat16}


@pytest.mark.parametrize("label", [-1, "K", 2 ** 31 - 1, -2 ** 31])
@pytest.mark.parametrize("form,dt,K", [("one launch", hb.BF16, 16), ("one launch", hb.F32, 12), ("stored", hb.BF16, 16), ("stored", hb.F32, 5),
                                       ("rows", hb.BF16, 1000), ("rows", hb.F32, 1001)])
def test_label_that_is_no_class(form, dt, K, label):
    B, M, Fx = 3, 7, 64
    label = K if label == "K" else label
    print(form, K, label, flush=True)
    g = torch.Generator().manual_seed(K)
    r = lambda *s: (torch.rand(s, generator=g) * 2 - 1).to(TDT[dt]).to(DEV)
    good = torch.randint(K, (B, M), generator=g, dtype=torch.int32)
    bad = good.clone()
    bad[1, 2] = label
    x, w, scores = r(B, M, Fx), r(B, Fx, K), r(B, M, K)
    ws = torch.empty(hb.softmax_xent_rows_workspace_bytes(B, M), dtype=torch.uint8, device=DEV)

    def loss_and_gradient(labels):
        z, d, loss = scores.clone(), torch.full((B, M, K), 9.0, dtype=TDT[dt], device=DEV), torch.zeros(B, device=DEV)
        if form == "one launch":
            hb.linear_xent(B, M, Fx, K, dt, x, w, None, z, labels.to(DEV), loss, d)
        elif form == "stored":
            hb.softmax_xent(B, M, K, dt, z, labels.to(DEV), loss, d)
        else:
            hb.softmax_xent_rows(B, M, K, dt, z, labels.to(DEV), loss, d, ws)
        return z, loss, d
    z, l0, d0 = loss_and_gradient(good)
    _, l1, d1 = loss_and_gradient(bad)
    assert torch.isfinite(l0).all() and torch.isnan(l1[1])
    assert torch.equal(l0[[0, 2]], l1[[0, 2]])
    other = torch.ones(B, M, dtype=torch.bool, device=DEV)
    other[1, 2] = False
    assert torch.equal(d0[other], d1[other])
    # one rounding to the storage type beside a few of fp32
    ref = torch.softmax(z[1, 2].double(), 0) / M
    assert ((d1[1, 2].double() - ref).abs() <= ref * (2.0 ** -8 if dt == hb.BF16 else 2.0 ** -18)).all()
