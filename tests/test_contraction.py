"""The one-pass and the segmented linear-attention prefill give the same bits
because both write out every fused multiply-add: where the compiler may
contract and where it may not, it emits the same arithmetic."""
import os
import re
import shutil
import subprocess
from collections import Counter

import pytest

from paper_2606_20537_amd import build as B

FILES = ["linattn_scan.hip", "linattn_seg.hip"]


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("hipcc is missing")
    out = tmp_path_factory.mktemp("asm")
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-shared")]
    procs = {}
    for f in FILES:
        for mode in ("fast", "off"):
            path = str(out / (f + "." + mode + ".s"))
            cmd = [B.HIPCC, *flags, "-ffp-contract=" + mode, "--cuda-device-only", "-S", "-I", os.path.join(B.ROOT, "include"),
                   "-I", B.CSRC, os.path.join(B.CSRC, f), "-o", path]
            procs[f, mode] = subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.PIPE, text=True), path
    result = {}
    for key, (proc, path) in procs.items():
        _, err = proc.communicate(timeout=300)
        assert proc.returncode == 0, err
        with open(path) as s:
            result[key] = Counter(re.findall(r"^\s(v_(?:fma|fmac|mad|mac|mul|add|sub|subrev)_f32)", s.read(), re.M))
    return result


@pytest.mark.parametrize("f", FILES)
def test_same_arithmetic(counts, f):
    assert counts[f, "fast"]["v_fma_f32"] > 0
    assert counts[f, "fast"] == counts[f, "off"]
