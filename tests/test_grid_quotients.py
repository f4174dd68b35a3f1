"""The exhaustive comparisons behind the quantizers' one product for rows of fp16 values and their scales without a division:
tests/host/grid_quotients.cpp, with the device's own functions. No GPU."""
import os
import subprocess

from paper_2603_22943_amd import build as B


def test_every_case(tmp_path):
    exe = str(tmp_path / "grid_quotients")
    root = os.path.dirname(B.HERE)
    r = subprocess.run([B.hipcc_path(), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-pthread",
                        "-I", os.path.join(root, "include"), "-I", B.CSRC, os.path.join(root, "tests", "host", "grid_quotients.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "grid_quotients: ok" in r.stdout, r.stderr[-3000:]
