"""The dealing of a launch's work to the XCDs, and the rule that counts the rounds it leaves them: tests/host/xcd_share.cpp. No GPU."""
import os
import subprocess

from paper_2603_22943_amd import build as B


def test_every_xcd_has_an_eighth(tmp_path):
    exe = str(tmp_path / "xcd_share")
    root = os.path.dirname(B.HERE)
    r = subprocess.run([B.hipcc_path(), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-I", os.path.join(root, "include"),
                        "-I", B.CSRC, os.path.join(root, "tests", "host", "xcd_share.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "xcd_share: ok" in r.stdout, r.stderr[-2000:]
