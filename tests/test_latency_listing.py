"""The least-squares residual kernel of a worker that fits a workgroup loads the sample's parameters ahead of its draws and uses
them behind: in the compiler's listing no wait for a vector load may stand in front of the draws' first logarithm."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2310_14423_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def test_parameters_are_not_waited_for_before_the_draws(tmp_path):
    out = tmp_path / "linreg.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-Wall", "-Wno-unused-function")]
    subprocess.run(["hipcc"] + flags + ["-I", build.INCLUDE, "-I", build.CSRC, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "grad_linreg.hip"), "-o", str(out)], check=True, capture_output=True, timeout=300)
    kernels = re.findall(r"^(_ZN3qsr\d+linreg_residual_row_kernel\w*):.*?$(.*?)^\s*s_endpgm", out.read_text(), re.S | re.M)
    assert kernels
    for name, body in kernels:
        head = body[:body.index("v_log_f32")]
        assert "global_load" in head and not re.search(r"s_waitcnt[^\n]*vmcnt", head), name
