"""The dual-time sweep of large 2D grids keeps its values in registers: the
compiler's report of the FP32 kernel at its widest tile (bounded to 128 vector
registers, four waves per SIMD) shows no spills."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_39474_amd", "csrc")

SRC = """
#include "msc_sweep_launch.h"
void go(const msc::SweepArgs<float, float>& A) {
  msc::launch_sweep_mode<msc::D2Q9, float, float, 256, 1, 256, msc::SW_DTS>(A, 1, nullptr, nullptr, nullptr);
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_fp32_sweep_does_not_spill(tmp_path):
    from paper_2609_39474_amd import build

    src = str(tmp_path / "sweep.hip")
    with open(src, "w") as f:
        f.write(SRC)
    r = subprocess.run([build.HIPCC] + build.COMMON + ["-I", CSRC, "--offload-device-only", "-c",
                                                       "-Rpass-analysis=kernel-resource-usage", src, "-o",
                                                       str(tmp_path / "sweep.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = re.findall(r"Function Name: (\S+).*?VGPRs Spill: (\d+)", r.stderr, flags=re.S)
    sweeps = [(n, int(v)) for n, v in found if "7k_sweepI" in n]
    assert len(sweeps) == 1, found
    assert sweeps[0][1] == 0, sweeps
