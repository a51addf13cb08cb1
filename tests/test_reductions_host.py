"""What the reductions rest on, checked on the CPU (their bits and their buffers): small
host programs compiled against the library's own headers.  Nothing runs on a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("name", ["row_sum_check", "partials_check"])
def test_host_program(tmp_path, name):
    exe = str(tmp_path / name)
    inc = [os.path.join(ROOT, "paper_2502_03249_amd", "csrc"), os.path.join(ROOT, "include")]
    cmd = [HIPCC, "-x", "hip", "-std=c++17", "-O1", "-ffp-contract=off", "--offload-arch=gfx950", "-Xclang",
           "-target-feature", "-Xclang", "-packed-fp32-ops"] + [f"-I{d}" for d in inc]
    r = subprocess.run(cmd + [os.path.join(ROOT, "tests", name + ".hip"), "-o", exe], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "bad 0" in r.stdout, r.stdout[-3000:]
