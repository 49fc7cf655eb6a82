"""The ctypes views of tests/plans.py against the structs of csrc/ops.h."""
import os
import subprocess

import pytest

from tests import plans

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_struct_layouts(tmp_path):
    lines, want = [], []
    for name, s in plans.STRUCTS.items():
        lines.append(f'printf("%zu\\n", sizeof(aj::{name}));')
        want.append(plans.C.sizeof(s))
        for f, _ in s._fields_:
            lines.append(f'printf("%zu\\n", offsetof(aj::{name}, {f}));')
            want.append(getattr(s, f).offset)
    src = tmp_path / "layout.cpp"
    src.write_text('#include <cstddef>\n#include <cstdio>\n#include "ops.h"\nint main() {\n' +
                   "\n".join(lines) + "\n}\n")
    exe = str(tmp_path / "layout")
    subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "-Wno-invalid-offsetof",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2606_04484_amd", "csrc"), "-x", "hip", str(src),
                    "-o", exe], check=True, cwd=str(tmp_path))
    got = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()
    assert [int(x) for x in got] == want
