"""The selection may be captured at any shape once a device has seen any first call of it: nothing in its launches asks the runtime
for a kernel attribute. CPU only: the host part is compiled, nothing runs."""
import os
import shutil
import subprocess

import pytest

from paper_2406_00023_amd import build


def undefined_symbols(source, directory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj = os.path.join(directory, "host.o")
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([hipcc, *flags, "--cuda-host-only", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-c",
                    os.path.join(build.CSRC, source), "-o", obj], check=True, capture_output=True)
    return subprocess.run(["nm", "-C", "-u", obj], check=True, capture_output=True, text=True).stdout


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_selection_sets_no_kernel_attribute(tmp_path):
    needed = undefined_symbols("select.hip", str(tmp_path))
    assert "hipLaunchKernel" in needed                   # (the list is that of the launches)
    assert "ensure_dynamic_lds" not in needed and "hipFuncSetAttribute" not in needed
