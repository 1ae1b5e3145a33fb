"""bench.py's line on stdout: the contract's fields whole, and short enough for a reader of the last kilobytes whatever
the complete record holds.  Its per-kernel table: a row for every operator the arrays call, named as the kernels are."""
import glob
import json
import os
import re
import shutil
import subprocess

import pytest

import bench


def test_line_is_short_and_complete():
    leg = {"value": 123456.789012345, "unit": "samples/s", "ms_per_step": 1.2345678901234567, "dtype": "bf16", "data": "synthetic",
           "config": {"workload": "some_array_B8_bf16", "B": 8}, "kernels": {f"kernel_{k}": {"ms_per_step": 0.1} for k in range(200)}}
    out = dict(metric="m", n_gpus=1, steps=20, warmup=5, higher_is_better=True, scaling="weak", vs_baseline=None, **leg,
               workloads={n: dict(leg) for n in ("c0", "c2", "c3", "c4")}, operators=[{"op": "x" * 100}] * 60, operators_note="n" * 500)
    line = bench.brief_line(out)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config"):
        assert line[k] == out[k], k
    assert {n: w["value"] for n, w in line["workloads"].items()} == {n: leg["value"] for n in out["workloads"]}
    text = json.dumps(line)
    assert len(text) < 2000 and "\n" not in text
    assert "kernels" in out and "operators" in out                       # the record itself keeps everything


#: element-wise operators of a few microseconds a step, and what computes sizes
UNTRACED = {"adadelta_step_multi", "adam_step", "bce_logits_strided", "bn_apply_fwd", "dropout", "mse", "steplr"}


def test_every_operator_of_the_arrays_has_a_row():
    src = open(os.path.join(bench.ROOT, "paper_2102_02344_amd", "arrays.py")).read()
    names = {n for n in re.findall(r"\bhb\.([a-z]\w+)\b", src)
             if not n.endswith(("_bytes", "_floats", "_supported", "_gives_sums"))}
    assert names - set(bench.Tracer.SINGLE_KERNEL) == UNTRACED


def test_conv_bn_pool_row():
    B, Nb, Ci, Co, L = 6, 16, 512, 2048, 2500
    a = [B, Nb, Ci, Co, L, 1] + [object()] * 14 + [None]
    z = B * Nb * Co * L * 2
    assert bench.algorithmic_flops("conv1x1_bn_pool_fwd", a) == 2.0 * B * Nb * Ci * Co * L
    pooled = bench.algorithmic_bytes("conv1x1_bn_pool_fwd", a)
    assert pooled == (B * Nb * (Ci + Co) * L + B * Co * (Ci + 1)) * 2 + B * Nb * Co * 6
    label = bench.kernel_label("conv1x1_bn_pool_fwd", a)
    a[20] = object()
    assert bench.algorithmic_bytes("conv1x1_bn_pool_fwd", a) == pooled + 2 * z
    assert "bn_apply_maxpool_kernel" in bench.kernel_label("conv1x1_bn_pool_fwd", a) != label


def test_profiled_traffic_is_that_of_present_kernels():
    """The keys of the counters' summaries name kernels that there are and that the table names."""
    src = open(bench.__file__).read() + " bn_fwd_conv_kernel bn_bwd_conv_kernel"
    csrc = "".join(open(f).read() for f in glob.glob(os.path.join(bench.ROOT, "paper_2102_02344_amd", "csrc", "*")))
    for path in glob.glob(os.path.join(bench.ROOT, "profiles", "*_traffic.json")):
        for key in json.load(open(path)):
            for kernel in re.findall(r"\w+_kernel\b", key):
                assert kernel in csrc and (kernel in src or kernel[:-len("_kernel")] in bench.Tracer.SINGLE_KERNEL), (path, kernel)


def test_profiled_kernels_are_in_the_library():
    """The kernels that the tables under profiles/ name, template arguments and all, are those that the library holds."""
    lib = os.path.join(bench.ROOT, "paper_2102_02344_amd", "libhfta.so")
    if not os.path.exists(lib) or shutil.which("nm") is None:
        pytest.skip("needs the built library and nm")
    syms = subprocess.run(["nm", "-C", lib], capture_output=True, text=True, check=True).stdout
    have = set(re.findall(r"__device_stub__(\w+_kernel(?:<[^()]*>)?)\(", syms))
    named = set()
    for path in glob.glob(os.path.join(bench.ROOT, "profiles", "*.md")):
        # (rows of bench.py's entries go by families' names, without arguments)
        named |= {n for n in re.findall(r"`(\w+_kernel(?:<[^`]*>)?)` (?:\||\()", open(path).read()) if "<" in n or "traffic" not in path}
    assert len(named) > 80 and named <= have, sorted(named - have)
