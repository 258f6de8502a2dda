"""Block sizes of the Poisson passes by side (CPU, no GPU): 512 threads for the FP32 passes above
64^3 but for the pencils of many boxes of 128^3, which measured slower so; and every pass's LDS
head fits what the launch gives it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_04925_amd", "csrc")


def test_block_sizes(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    lines = ['#include "kernels_poisson.hip"', "namespace scola {"]
    for R in range(1, 9):
        usual = 256 if R < 5 else 512
        for name, size in (("pass_threads", usual),
                           ("many_pencils_threads", 256 if R == 8 else usual)):
            n = "%s<%%s, %d>()" % (name, R)
            lines += ["static_assert(%s == %d);" % (n % "float", size),
                      "static_assert(%s == 256);" % (n % "double"),
                      "static_assert(mfma_head<%s>() <= mfma_head<%d>());" % (n % "float", usual)]
    src = tmp_path / "block_sizes.hip"
    src.write_text("\n".join(lines + ["}"]))
    r = subprocess.run([hipcc, "-std=c++17", "--offload-arch=gfx950", "-fsyntax-only",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
