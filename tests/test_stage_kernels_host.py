"""The FP64 stage kernels compiled for the host and run thread by thread
(tests/native/stage_kernels_check.cpp): no dependence on the order of a
workgroup's waves and threads between barriers nor on unwritten LDS, the
axis-by-axis item and the 3-D lane kernel against the point-by-point item, and
the CFL rate of a last stage that stores in place against the stored state,
with partly filled workgroups of the lane kernel."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CXX = shutil.which("amdclang++") or "/opt/rocm/bin/amdclang++"


@pytest.mark.skipif(not os.path.exists(CXX), reason="amdclang++ not found")
@pytest.mark.parametrize("dim,p,sizes", [(2, 0, "2,6"), (2, 1, "2,6,16"), (2, 3, "6,12"), (3, 0, "2,4"), (3, 1, "2,4"), (3, 2, "2,4"), (3, 3, "2,4")])
def test_stage_kernels_on_the_host(dim, p, sizes, tmp_path):
    exe = str(tmp_path / "stage_kernels_check")
    cmd = [CXX, "-x", "c++", "-std=c++17", "-O1", "-mfma", "-w", "-fconstexpr-steps=200000000",
           "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(HERE, "native", "hostsim"), "-I" + os.path.join(ROOT, "include"),
           f"-DDG_D={dim}", f"-DDG_P={p}", "-DDG_SIZES={" + sizes + "}",
           os.path.join(HERE, "native", "stage_kernels_check.cpp"),
           os.path.join(ROOT, "paper_2502_12620_amd", "csrc", "forest.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(r.stdout[-3000:])
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert r.stdout.strip().splitlines()[-1].startswith("OK")
