"""Which kernels take a C = 1280 or 640 layer or batched call, against timings of all forms: tests/host/mid_rule.cpp on the CPU; on the GPU head
groups and stages give the same bits on either side of each line."""
import os
import subprocess

import numpy as np
import pytest

from paper_2603_22943_amd import build as B


def test_the_rule_takes_the_faster_kernels(tmp_path):
    exe = str(tmp_path / "mid_rule")
    root = os.path.dirname(B.HERE)
    r = subprocess.run([B.hipcc_path(), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(root, "include"),
                        "-I", B.CSRC, os.path.join(root, "tests", "host", "mid_rule.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "mid_rule: ok" in r.stdout, r.stderr[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("B,tiles,H,w_layout", [(1, 32, 8, 1), (1, 33, 8, 1), (4, 12, 8, 1), (1, 52, 8, 1), (1, 51, 20, 1), (4, 15, 20, 1), (1, 64, 20, 1),
                                                (1, 26, 20, 0), (1, 27, 20, 0), (2, 24, 20, 0), (1, 52, 20, 0)])
def test_both_give_the_same_bits(B, tiles, H, w_layout):
    from test_gpu_token_tiles import Layer

    L = Layer(B, 16 * tiles - 3, 1280, H, w_layout=w_layout)
    got = L.run()
    assert np.array_equal(got, L.run(tok_tile=16)) and np.array_equal(got, L.run(tok_tile=32))
