"""The scans read their arguments in one go: every pointer is loaded before the
first branch, not behind the exit of the workgroups without a head (a second
trip to memory on each launch, 5 % of a short call)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_20537_amd import build as B


@pytest.mark.parametrize("f, pointers, kernels", [("linattn_scan.hip", 8, 9), ("gdn_scan.hip", 10, 4)])
def test_loaded_before_the_first_branch(tmp_path, f, pointers, kernels):
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("hipcc is missing")
    path = str(tmp_path / "scan.s")
    flags = [x for x in B.FLAGS if x not in ("-fPIC", "-shared")]
    run = subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-S", "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC,
                          os.path.join(B.CSRC, f), "-o", path], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr
    with open(path) as s:
        bodies = re.findall(r"^(_ZN\S*_scan_kernel\S*):(.*?)^\.Lfunc_end", s.read(), re.M | re.S)
    assert len(bodies) == kernels
    for name, body in bodies:
        late = body[body.index("s_cbranch"):]
        at = [int(x, 0) for x in re.findall(r"s_load_dword\S*\s+\S+\s+s\[0:1\], (\S+)", late)]
        assert not [x for x in at if x < 8 * pointers], name
