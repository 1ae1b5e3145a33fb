"""Sums of split products' parts, four outputs a thread (2^19 outputs and more, whole 16-byte pieces) and one: the same bits, whatever
the number of parts, and what float64 gives."""
import pytest
import torch

from paper_2102_02344_amd import binding as hb

pytestmark = pytest.mark.gpu
DEV = "cuda"


# 1024 x 512 is the first output of 2^19, 1024 x 508 lies below, 1027 x 513 above but not in fours; 128 rows a part
@pytest.mark.parametrize("parts,Fx,Fy", [(p, 1024, 512) for p in (2, 3, 4, 5, 6, 7, 9, 16)] + [(5, 1024, 508), (5, 1027, 513), (3, 1028, 512)])
def test_parts_in_either_form(parts, Fx, Fy):
    B, M = 1, 128 * parts
    assert hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.F32) == parts * B * Fx * Fy * 4
    g = torch.Generator(device=DEV).manual_seed(parts)
    x, dy = (torch.randn(s, generator=g, device=DEV) for s in ((B, M, Fx), (B, M, Fy)))
    ws = torch.empty(hb.linear_bwd_workspace_bytes(B, M, Fx, Fy, hb.F32), dtype=torch.uint8, device=DEV)
    n, got = B * Fx * Fy, []
    for off in (0, 1):                                     # an output that starts off 16 bytes is summed one element a thread
        buf = torch.full((n + 9,), float("nan"), device=DEV)
        dw = buf[4 + off:4 + off + n].view(B, Fx, Fy)
        hb.linear_bwd(B, M, Fx, Fy, hb.F32, x, None, dy, None, dw, None, ws)
        assert torch.isnan(buf[:4 + off]).all() and torch.isnan(buf[4 + off + n:]).all()
        got.append(dw.clone())
    assert torch.equal(got[0].view(torch.int32), got[1].view(torch.int32))
    ref, mag = x[0].t().double() @ dy[0].double(), x[0].t().double().abs() @ dy[0].double().abs()
    # products of operands in three bf16 parts and fp32 sums: 2^-23 of each of the sum's M terms at the most
    assert ((got[0][0].double() - ref).abs() <= M * 2.0 ** -23 * mag).all()
    assert float((got[0][0].double() - ref).norm() / ref.norm()) <= 2.0 ** -21
