"""The selection kernel's scalar registers, as the compiler reports them: two of
its sixteen-wave workgroups share a compute unit only if eight waves of them fit
a SIMD's 800, each with the 16 that the trap handler takes."""
import os
import re
import subprocess

from paper_2608_04771_amd import build


def test_two_workgroups_fit_a_compute_unit():
    cmd = [build._hipcc(), "-x", "hip", f"--offload-arch={build.ARCH}", "-O3", "-std=c++17", "--cuda-device-only",
           f"-I{os.path.join(build.ROOT, 'include')}", *build.NO_PACKED_FP32,
           "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(build.CSRC, "select_compact.hip"),
           "-o", os.devnull]
    out = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True).stdout
    kernel = out[out.index("select_kernel"):]
    num = {k: int(re.search(rf"{k}[^:]*: (\d+)", kernel).group(1)) for k in ("TotalSGPRs", "VGPRs", "LDS Size")}
    per_wave = (num["TotalSGPRs"] + 15) // 16 * 16 + 16
    assert 8 * per_wave <= 800, num
    assert num["VGPRs"] <= 64 and 2 * num["LDS Size"] <= 160 * 1024, num
