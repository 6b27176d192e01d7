"""The one-pass search keeps a row's candidates as 64 bits per lane, which holds up to the largest supported number of key blocks.
Raising that limit alone must not build."""
import os
import shutil
import subprocess

import pytest

from paper_2603_06199_amd import build as hip_build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.parametrize("limit,builds", ((4096, True), (4097, False)))
def test_limit(tmp_path, limit, builds):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("needs hipcc")
    csrc = tmp_path / "package" / "csrc"
    shutil.copytree(hip_build.CSRC, csrc)
    shutil.copytree(os.path.join(hip_build.HERE, "..", "include"), tmp_path / "include")
    seen = 0
    for f in os.listdir(csrc):
        text = (csrc / f).read_text()
        seen += text.count("kMaxBlocksPerSeq = 4096;")
        (csrc / f).write_text(text.replace("kMaxBlocksPerSeq = 4096;", f"kMaxBlocksPerSeq = {limit};"))
    assert seen == 1
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-O3")]
    r = subprocess.run([HIPCC] + flags + ["--cuda-device-only", "-fsyntax-only"] + [str(csrc / s) for s in hip_build.SOURCES],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == builds, r.stderr[-2000:]
    assert builds or "static assertion failed" in r.stderr
