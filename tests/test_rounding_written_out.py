"""Kernels of which several forms must give the same bits (a step launched directly or
in a window, the row kernels and the row-block kernel) leave no rounding to what the
compiler contracts: built with and without contraction they have the same additions,
multiplications and fused ones."""

import collections
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2507_18969_amd import build as B

KINDS = {"v_add_f32": "add", "v_sub_f32": "add", "v_subrev_f32": "add", "v_mul_f32": "mul", "v_fma_f32": "fma",
         "v_fmac_f32": "fma", "v_fmamk_f32": "fma", "v_fmaak_f32": "fma"}


def _counts(src, out, *flags):
    """kernel -> counts of its FP32 additions, products and fused ones."""
    cmd = [B.HIPCC, *B.FLAGS, *flags, "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    got, cur = {}, None
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            cur = got.setdefault(m.group(1), collections.Counter())
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None and (m := re.match(r"\t(v_\w+?_f32)(_e32|_e64|_dpp|_e64_dpp)?\s", line)):
            if m.group(1) in KINDS:
                cur[KINDS[m.group(1)]] += 1
    return got


@pytest.mark.parametrize("src,kernels,loose", [
    ("kernels.hip", ["fdm_fwd_kernel", "fdm_bwd_kernel", "ln_fwd_256_kernel", "ln_bwd_256_kernel", "adam_kernel",
                     "colsum_partial_kernel"], 0),
    ("wgrad_adam.hip", ["wgrad_adam_kernel"], 0),
    ("gemm_fp32.hip", ["gemm_fp32_kernel", "wgrad_fp32_kernel"], 0),
    # (the loss's logarithm, which the compiler expands: one operation, in head_kernel too)
    ("fused_fp32.hip", ["fused_fp32_kernel"], 1)])
def test_contraction_changes_nothing(tmp_path, src, kernels, loose):
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not available")
    with ThreadPoolExecutor(2) as ex:
        a, b = ex.map(lambda f: _counts(src, tmp_path / f"{len(f)}.s", *f), [(), ("-ffp-contract=off",)])
    for k in kernels:
        names = [n for n in a if f"{len(k)}{k}" in n]
        assert names, k
        for n in names:
            assert abs(a[n]["fma"] - b[n]["fma"]) <= loose and a[n]["mul"] == b[n]["mul"], (n, a[n], b[n])
