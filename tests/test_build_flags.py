"""The library's compiler flags refuse a function that ends without its return value (host code, no device use)."""
import os
import shutil
import subprocess

import pytest

from paper_1105_0542_amd import build


@pytest.mark.skipif(not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")), reason="no hipcc")
@pytest.mark.parametrize("body,ok", [("return x;", True), ("", False), ("if (x) return 1;", False)])
def test_missing_return_does_not_compile(tmp_path, body, ok):
    src = tmp_path / "f.hip"
    src.write_text("template <int K> int f(int x) { %s }\ntemplate int f<1>(int);\n" % body)
    r = subprocess.run([build.hipcc()] + build.HIP_FLAGS + ["--cuda-host-only", "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == ok, r.stderr
