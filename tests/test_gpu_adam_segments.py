"""One Adam launch over a parameter-major arena whose segments have any length: groups of four that lie in one model's part,
that cross from one model or segment to the next, arenas shorter than a workgroup and with a last group of fewer than four,
and arrays that are only element-aligned.  Same reference and tolerance as the per-model operator."""
import numpy as np
import pytest
import torch

import hfta_inputs as hi
from oracle import array as oa
from test_gpu_ops import DT, dev, empty, host
from util import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gdtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("B,sizes", [(3, (1, 9, 50, 977)), (5, (2, 1)), (2, (4096, 3, 4096, 1030)), (7, (341,)), (4, (64, 4, 1024, 8))])
def test_segments_of_any_length(B, sizes, shift, gdtype):
    from paper_2102_02344_amd import binding as hb
    print(f"adam segments B={B} {sizes} shift={shift} {gdtype}", flush=True)
    off = tuple(int(x) for x in np.concatenate([[0], np.cumsum(sizes)]))
    total = B * off[-1]
    hp = hi.adam_hparams(55, B)
    H = {k: dev(a) for k, a in hp.items()}
    th0, g = hi.normal(56, (total,)) * 0.1, hi.normal(57, (total,), gdtype)
    bufs = [empty((total + 1,), torch.float32)[shift:][:total] for _ in range(3)]
    G = empty((total + 1,), gdtype)[shift:][:total]
    LP = empty((total + 1,), torch.bfloat16)[shift:][:total]
    TH, M_, V_ = bufs
    TH.copy_(dev(th0)); M_.zero_(); V_.zero_(); G.copy_(dev(g, gdtype))
    for t in (1, 2):
        hb.adam_step_multi(B, off, DT[gdtype], TH, G, M_, V_, LP, H["lr"], H["beta1"], H["beta2"], H["eps"], H["wd"], t, 1)
    th, m, v = th0.copy(), np.zeros(total, np.float32), np.zeros(total, np.float32)
    for j, n in enumerate(sizes):
        s = slice(B * off[j], B * off[j + 1])
        a = [x[s].reshape(B, n) for x in (th, g, m, v)]
        for t in (1, 2):
            a[0], a[2], a[3] = oa.adam_step(B, a[0], a[1], a[2], a[3], hp["lr"], hp["beta1"], hp["beta2"], hp["eps"], hp["wd"], t, True)
        check(host(TH)[s], a[0].reshape(-1), 1e-5, f"theta {j}")
        check(host(M_)[s], a[2].reshape(-1), 1e-5, f"m {j}")
        check(host(V_)[s], a[3].reshape(-1), 1e-5, f"v {j}")
    assert torch.equal(LP, TH.to(torch.bfloat16))


@pytest.mark.parametrize("gdtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,sizes", [(3, (9, 320000, 50, 977, 1)), (5, (2, 187283, 1, 1)), (2, (4096, 463215, 30)), (256, (3585,)),
                                     (3, (308130, 1, 8)), (3, (308130, 1, 7)), (40, (31, 33000, 2, 3))])
def test_large_arenas_of_odd_segments(B, sizes, gdtype):
    """The same in arenas large enough to be taken in groups of four (from 917504 elements and 768 more per part on, of more
    than 128 models from 917504); the two of 308130 lie on either side."""
    test_segments_of_any_length(B, sizes, 0, gdtype)
