"""Codes whose quotient lies exactly between two integers, which the quantizers settle several dwords at a time: rows of odd integers
beside a largest value of 254 (x * 127 / 254 = x / 2), one such value per row, and rows of nothing else."""
import numpy as np
import pytest
import torch

from oracle import taq_oracle as O
from paper_2603_22943_amd import synth
from tests import gpu_helpers as G
from paper_2603_22943_amd import taq as T

pytestmark = pytest.mark.gpu


def tie_rows(rows, cols, seed, share):
    rng = np.random.Generator(np.random.PCG64(seed))
    odd = 2 * rng.integers(-126, 127, size=(rows, cols)) + 1          # ties: x / 2 is a half
    even = 2 * rng.integers(-127, 128, size=(rows, cols))
    x = np.where(rng.random((rows, cols)) < share, odd, even)
    x[np.arange(rows), rng.integers(0, cols, size=rows)] = 254 * rng.choice((-1, 1), size=rows)
    return x.astype(np.float16)


@pytest.mark.parametrize("cols", [8, 64, 320, 520, 1024, 1032, 2048, 2056])
@pytest.mark.parametrize("share", [0.002, 0.5, 1.0])
def test_weight_codes(cols, share):
    W = tie_rows(37, cols, cols, share)
    code, scale = T.taq_quantize_weight(G.dev(W))
    want, s = O.quantize_weight(W)
    assert np.array_equal(code.cpu().numpy(), want) and np.array_equal(scale.cpu().numpy(), s.reshape(-1))


@pytest.mark.parametrize("C,H,N,w_layout", [(320, 8, 45, 1), (640, 8, 33, 0), (640, 10, 20, 1), (1280, 8, 19, 0), (1280, 20, 33, 1), (96, 4, 50, 0)])
@pytest.mark.parametrize("share", [0.002, 1.0])
def test_hidden_codes_and_the_block(C, H, N, w_layout, share):
    L = synth.make_layer("ties", seed=C + N, B=2, N=N, C=C, H=H, Cc=64, T=77, bits_kv=8, trigger_positions=(3,), trigger_scale=3.0)
    hidden = tie_rows(2 * N, C, C + N, share).reshape(2, N, C)
    g = G.GpuRun(L, hidden=hidden, w_layout=w_layout)
    want, scale = O.symq(hidden, 8)
    assert np.array_equal(g.taps["h_code"].reshape(want.shape), want)
    assert np.array_equal(g.taps["s_h"].reshape(-1), np.asarray(scale, dtype=np.float32).reshape(-1))
    quick = G.GpuRun(L, hidden=hidden, w_layout=w_layout, taps=False)  # the build without taps: a fixed number of text tiles
    assert np.array_equal(quick.out.view(np.uint16), g.out.view(np.uint16))
