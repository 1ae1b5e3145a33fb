"""Residual LayerNorm forward: the one call against the element-wise sum followed by LayerNorm, which it has to
match bit for bit, at rows of one lane's piece, half a wavefront, a whole one, two pieces per lane, rows past
the register-resident form, and row counts that leave a workgroup's last slots empty."""
import pytest
import torch

import hfta_inputs as hi
from util import DT, TDT, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,R,E", [(2, 3, 8), (3, 37, 256), (2, 9, 264), (1, 1, 512), (2, 65, 520), (2, 5, 1032), (2, 7, 30)])
def test_add_layernorm_is_add_then_layernorm(dtype, B, R, E):
    from paper_2102_02344_amd import binding as hb
    x1, x2 = (dev(hi.normal(s, (B, R, E), dtype), dtype) for s in (601, 602))
    w, b = (dev(hi.normal(s, (B, E)).astype("float32")) for s in (603, 604))
    new = lambda: [torch.full((B, R, E), float("nan"), dtype=TDT[dtype], device="cuda") for _ in range(2)]
    st = lambda: [torch.full((B * R,), float("nan"), device="cuda") for _ in range(2)]
    (s0, y0), (m0, i0), (s1, y1), (m1, i1) = new(), st(), new(), st()
    hb.add(B * R * E, DT[dtype], x1, x2, s0)
    hb.layernorm_fwd(B, R, E, DT[dtype], s0, w, b, 1e-5, m0, i0, y0)
    hb.add_layernorm_fwd(B, R, E, DT[dtype], x1, x2, s1, w, b, 1e-5, m1, i1, y1)
    for a, c in ((s0, s1), (y0, y1), (m0, m1), (i0, i1)):
        assert torch.equal(a, c) and bool(torch.isfinite(a).all())


@pytest.mark.parametrize("R", [8191, 8193, 16385, 20011])
@pytest.mark.parametrize("E", [64, 66])
def test_backward_of_many_rows(R, E):
    """Column sums over more rows than 128 workgroups of 16 hold (register-resident and plain rows), at counts that leave
    the last workgroup short: against float64 of the same values.  R terms of at most 4 roundings each on the way in, added
    in chains: a term's error is below (4 + R / 128) 2^-24 of it in any of the orders."""
    from paper_2102_02344_amd import binding as hb
    B = 1
    x, dy = dev(hi.normal(611, (B, R, E))), dev(hi.normal(612, (B, R, E)))
    w, b = dev(hi.normal(613, (B, E)).astype("float32")), dev(hi.normal(614, (B, E)).astype("float32"))
    mean, inv, y, dx = (torch.empty(s, device="cuda") for s in ((R,), (R,), (B, R, E), (B, R, E)))
    hb.layernorm_fwd(B, R, E, 0, x, w, b, 1e-5, mean, inv, y)
    dw, db = torch.full((B, E), float("nan"), device="cuda"), torch.full((B, E), float("nan"), device="cuda")
    ws = torch.empty(hb.layernorm_bwd_workspace_bytes(B, R, E), dtype=torch.uint8, device="cuda")
    hb.layernorm_bwd(B, R, E, 0, x, dy, w, mean, inv, dx, dw, db, ws)
    xh = (x.double()[0] - mean.double()[:, None]) * inv.double()[:, None]
    for got, term in ((dw, dy.double()[0] * xh), (db, dy.double()[0])):
        lim = (4 + R / 128) * 2.0 ** -24 * term.abs().sum(0)
        assert bool(((got[0].double() - term.sum(0)).abs() <= lim).all())
