"""Embedding rows and their gradients where ids repeat as in real text and padding, and rows past 256 columns.

The gradient of a table row is scale * (the fp32 sum of its positions' gradient rows in increasing order), so the
reference is that sum, in numpy's fp32, and has to be met bit for bit: an id met once, up to as many rows as a wavefront
has in flight (8), past that (9, 16, 17 and half of all positions), more positions than one search step (512), the most
positions the operator takes, columns around 64 and 256, and few positions under many columns."""
import numpy as np
import pytest
import torch

import hfta_inputs as hi
from util import DT, TDT, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    from paper_2102_02344_amd import binding
    return binding


def ids(kind, B, R, V):
    g = np.random.default_rng(31)
    if kind == "uniform":
        return g.integers(0, V, (B, R)).astype(np.int32)
    if kind == "padded":                     # the second half of every model's positions holds one id
        i = g.integers(0, V, (B, R))
        i[:, R // 2:] = V - 1
        return i.astype(np.int32)
    if kind == "counts":                     # ids met 1, 2, .. times, in a shuffled order
        i = np.repeat(np.arange(V), np.arange(1, V + 1))
        return np.stack([g.permutation(np.resize(i, R)) for _ in range(B)]).astype(np.int32)
    return np.zeros((B, R), np.int32)        # one id


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind,B,R,V,E", [
    ("counts", 2, 300, 24, 64), ("counts", 1, 153, 17, 257), ("padded", 2, 1100, 300, 72), ("padded", 1, 2048, 900, 520),
    ("one", 2, 513, 5, 65), ("one", 1, 1, 3, 1030), ("uniform", 1, 16, 9, 2048), ("uniform", 3, 700, 1000, 256),
    ("padded", 1, 7680, 1000, 40)])
def test_rows_and_gradients(hb, dtype, kind, B, R, V, E):
    print(kind, dtype, B, R, V, E, flush=True)
    idx = ids(kind, B, R, V)
    table, pos, dy = hi.normal(731, (B, V, E), dtype), hi.normal(732, (R, E)).astype(np.float32), hi.normal(733, (B, R, E), dtype)
    I = dev(idx)
    Y = torch.full((B, R, E), float("nan"), dtype=TDT[dtype], device="cuda")
    hb.embedding_fwd(B, R, V, E, DT[dtype], dev(table, dtype), I, 2.0, dev(pos), R, Y)
    ref = torch.from_numpy(np.stack([np.float32(2.0) * table[b][idx[b]].astype(np.float32) + pos for b in range(B)])).to(TDT[dtype])
    assert torch.equal(Y.cpu(), ref)                     # (2 x is exact: one rounding either way)
    dT = torch.full((B, V, E), float("nan"), device="cuda")
    hb.embedding_bwd(B, R, V, E, DT[dtype], dev(dy, dtype), I, 1.5, dT)
    acc = np.zeros((B, V, E), np.float32)
    for b in range(B):
        for r in range(R):
            acc[b, idx[b, r]] += dy[b, r].astype(np.float32)
    assert np.array_equal(dT.cpu().numpy(), np.float32(1.5) * acc)


def test_a_frequent_id_is_no_serial_chain(hb):
    """Half of all positions on one id cost a small multiple of uniformly drawn ids, whatever the columns: 2.7 and 3.0
    times here.  One wavefront walking the rows one by one took 36 times in the first of the two."""
    for B, R, V, E in ((8, 2048, 8192, 256), (1, 4096, 1000, 512)):
        dy, dT = torch.ones(B, R, E, dtype=torch.bfloat16, device="cuda"), torch.empty(B, V, E, device="cuda")
        us = []
        for kind in ("uniform", "padded"):
            I = dev(ids(kind, B, R, V))
            call = lambda: hb.embedding_bwd(B, R, V, E, 1, dy, I, 1.0, dT)
            for _ in range(3):
                call()
            times = []
            for _ in range(9):
                a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(5):
                    call()
                z.record()
                torch.cuda.synchronize()
                times.append(a.elapsed_time(z) * 200)
            us.append(sorted(times)[4])
        print(f"{B} x {R} x {E}: uniform {us[0]:.1f} us, padded {us[1]:.1f} us", flush=True)
        assert us[1] < 10 * us[0]
