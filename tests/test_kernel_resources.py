"""The attention kernels keep everything in registers: a kernel that spills pays for
scratch memory on every step.  Read from the compiler's resource remarks for the
library's own build options (nothing is run)."""
import os
import re
import subprocess

import pytest

from paper_2606_04484_amd import build

SRC = "attention_mfma.hip"


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not installed")
def test_attention_kernels_use_no_scratch(tmp_path):
    r = subprocess.run([build.HIPCC, *build.FLAGS, *build.FILE_FLAGS[SRC], "-x", "hip",
                        "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, SRC), "-o", str(tmp_path / "x.o")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    scratch = dict(re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", r.stderr,
                              re.S))
    assert sum("mfma" in k for k in scratch) >= 10
    assert {k: v for k, v in scratch.items() if v != "0"} == {}
