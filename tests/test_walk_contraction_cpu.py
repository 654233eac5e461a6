"""The analog walk's arithmetic is the same whether or not the compiler fuses multiplies and adds by
itself: the equality of its regimes (a lane to a walk, lane groups) does not rest on that choice.
The walk kernels' code is compiled both ways and their FP32 instructions are counted; a multiply that
is fused in one of them only shows as one multiply less.  (Additions count with the fused ones: the
compiler's own expansion of expf, taken once at a walk's start, trades one for the other.)"""
import collections
import os
import re
import subprocess

import pytest

from paper_2512_13965_amd import _build

OPS = re.compile(r"^\s+v_(fma|fmac|fmaak|fmamk|mul|add|sub|subrev|mac|mad|dot2c|rcp|sqrt|log|sin|cos|exp)_f32")


def _counts(tmp_path, contract):
    out = str(tmp_path / f"{contract}.s")
    subprocess.run([_build.HIPCC, *_build.FLAGS, f"-ffp-contract={contract}", "-x", "hip", "--cuda-device-only", "-S",
                    os.path.join(_build.CSRC, "gmc_walk.hip"), "-o", out], check=True, capture_output=True)
    kernels, name = collections.defaultdict(collections.Counter), None
    for line in open(out):
        m = re.match(r"^(_Z\S+):", line)
        if m:
            name = m.group(1)
        m = OPS.match(line)
        if m and name and "walk_kernel" in name:
            op = m.group(1)
            op = "add" if op.startswith(("fma", "add", "sub")) else op
            kernels[name][op] += 1
    return kernels


def test_walk_kernels_do_not_depend_on_contraction(tmp_path):
    if not os.path.exists(_build.HIPCC):
        pytest.skip("no hipcc")
    fast, off = _counts(tmp_path, "fast"), _counts(tmp_path, "off")
    assert len(fast) == 4 and all(c["add"] > 100 for c in fast.values())
    assert fast == off
