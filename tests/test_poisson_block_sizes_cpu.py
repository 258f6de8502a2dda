"""Block sizes of the Poisson passes, by side and pass (CPU, no GPU): 512 threads for the FP32
passes above 64^3 but for the pencils of 128^3, which measured slower so; and every pass's LDS
head fits what the launch gives it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_04925_amd", "csrc")


def want(R, p):
    return 256 if R < 5 or (p == 2 and R == 8) else 512


def test_block_sizes(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    lines = ['#include "kernels_poisson.hip"', "namespace scola {"]
    for R in range(1, 9):
        for p in (1, 2, 3):
            n = "pass_threads<%%s, %d, %d>()" % (R, p)
            lines += ["static_assert(%s == %d);" % (n % "float", want(R, p)),
                      "static_assert(%s == 256);" % (n % "double"),
                      "static_assert(mfma_head<%s>() <= mfma_head<%d>());"
                      % (n % "float", 512 if R >= 5 else 256)]
    src = tmp_path / "block_sizes.hip"
    src.write_text("\n".join(lines + ["}"]))
    r = subprocess.run([hipcc, "-std=c++17", "--offload-arch=gfx950", "-fsyntax-only",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
