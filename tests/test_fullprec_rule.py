"""Which kernels the full-precision path and the token sweep take, against timings of the forms: tests/host/fullprec_rule.cpp. No GPU."""
import os
import subprocess

from paper_2603_22943_amd import build as B


def test_the_rules_take_the_faster_kernels(tmp_path):
    exe = str(tmp_path / "fullprec_rule")
    root = os.path.dirname(B.HERE)
    r = subprocess.run([B.hipcc_path(), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(root, "include"),
                        "-I", B.CSRC, os.path.join(root, "tests", "host", "fullprec_rule.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "fullprec_rule: ok" in r.stdout, r.stderr[-4000:]
