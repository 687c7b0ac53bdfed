"""What the compiler made of two kernels whose speed hangs on it, from its listings."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2310_14423_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def _listing(name, tmp_path):
    out = tmp_path / "listing.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-Wall", "-Wno-unused-function")]
    subprocess.run(["hipcc"] + flags + ["-I", build.INCLUDE, "-I", build.CSRC, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, name), "-o", str(out)], check=True, capture_output=True, timeout=300)
    return out.read_text()


def test_parameters_are_not_waited_for_before_the_draws(tmp_path):
    """The least-squares residual kernel of a worker that fits a workgroup loads the sample's parameters ahead of its draws and
    uses them behind: no wait for a vector load in front of the draws' first logarithm."""
    kernels = re.findall(r"^(_ZN3qsr\d+linreg_residual_row_kernel\w*):.*?$(.*?)^\s*s_endpgm", _listing("grad_linreg.hip", tmp_path), re.S | re.M)
    assert kernels
    for name, body in kernels:
        head = body[:body.index("v_log_f32")]
        assert "global_load" in head and not re.search(r"s_waitcnt[^\n]*vmcnt", head), name


def test_lds_of_the_fp32_products(tmp_path):
    """The launch of two gradients holds no more LDS than one of them: 24 KiB with two groups of wavefronts."""
    sizes = re.findall(r"\.amdhsa_kernel (_ZN3qsr\d+sgemm_\w+)\s+\.amdhsa_group_segment_fixed_size (\d+)", _listing("grad_mlp2.hip", tmp_path))
    assert len(sizes) >= 4 and any("pair" in name for name, _ in sizes)
    assert all(int(size) <= 24 * 1024 for _, size in sizes), sizes
