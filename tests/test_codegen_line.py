"""The code-generation guard of test_codegen.py over the line-evaluating chain kernel and the
iteration kernels."""
import subprocess

import pytest
import test_codegen as T


@pytest.mark.parametrize("source", ["nss_line.hip", "nss_iter.hip"])
def test_no_select_on_stale_condition_code(tmp_path, source):
    out = tmp_path / "k.s"
    r = subprocess.run(["hipcc", "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only",
                        "-S", "-o", str(out), T.CSRC + "/" + source],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    assert T.suspicious_selects(out.read_text()) == []
