"""launch_kernel checks a launch's arguments as a call would: what does not convert to the kernel's parameters does not compile."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_12574_amd", "csrc")

SOURCE = """#include "hi_device.h"
__global__ void kernel(const float* x, long n, int* y);
void launch(float* x, int* y, long n) { hi::launch_kernel(kernel, dim3(1), dim3(64), 0, nullptr, nullptr, ARGS); }
"""


@pytest.mark.parametrize("args,compiles", [("x, n, y", True), ("x, 3, nullptr", True), ("y, n, x", False), ("x, n, n", False),
                                           ("x, x, y", False), ("x, n", False)])
def test_launch_arguments(tmp_path, args, compiles):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    from paper_2502_12574_amd.build import HIPCC_FLAGS
    src = tmp_path / "launch.hip"
    src.write_text(SOURCE.replace("ARGS", args))
    r = subprocess.run([hipcc, *HIPCC_FLAGS, "-x", "hip", "-I", CSRC, "-fsyntax-only", str(src)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert (r.returncode == 0) == compiles, r.stdout[-2000:]
