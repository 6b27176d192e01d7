"""No kernel of the library needs scratch memory: compute calls allocate nothing, and scratch would be the runtime's to provide at a
launch.  Read off the resource notes in the assembly the compiler makes of all of them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_06199_amd import build as hip_build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_no_scratch_no_spills(tmp_path):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("needs hipcc")
    out = tmp_path / "flashprefill.s"
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
    subprocess.run([HIPCC] + flags + ["--cuda-device-only", "-S", "-o", str(out)] +
                   [os.path.join(hip_build.CSRC, s) for s in hip_build.SOURCES], check=True, capture_output=True)
    notes = out.read_text().split("amdhsa.kernels:")[1].split("\namdhsa.")[0]
    kernels = re.split(r"^  - ", notes, flags=re.M)[1:]
    found = {}
    for k in kernels:
        get = lambda key: re.search(rf"\.{key}:\s*(\S+)", k).group(1)
        found[get("symbol")] = (int(get("private_segment_fixed_size")), int(get("vgpr_spill_count")))
    # 10 attention kernels, 4 with two waves per 32 queries, 20 of the search, 5 of pooling, 2 of the threshold
    assert len(found) == 41, sorted(found)
    assert not {k: v for k, v in found.items() if v != (0, 0)}
