"""Build options of the library's dispatch, on the CPU: the host code is
compiled with the option and the kernels it can launch are listed."""
import os
import subprocess

import pytest

from paper_1809_02390_amd import build

MANY = ("stepk_kernel", "step2_kernel", "march_kernel")


# the host half of the kernels' source only (a few seconds)
@pytest.mark.parametrize("fuse", [0, 1])
def test_fuse_steps_option(tmp_path, fuse):
    """-DLBM_FUSE_STEPS=0 leaves no kernel of several steps in the library;
    with 1, the default, every one is there."""
    obj = str(tmp_path / "kernels.o")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--offload-host-only", "-c",
                    f"-DLBM_FUSE_STEPS={fuse}", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(build.CSRC, "lbm_kernels.hip"), "-o", obj], check=True, capture_output=True)
    names = subprocess.run(["nm", obj], check=True, capture_output=True, text=True).stdout
    assert [k in names for k in MANY] == [bool(fuse)] * 3
    assert "step_kernel" in names
