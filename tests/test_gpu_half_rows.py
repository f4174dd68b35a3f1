"""Codes of fp16 rows, which one product settles unless 127 divides the significand of the row's largest value: rows of every kind of significand,
values of exactly half the largest (the only quotient, 63.5, that lies between two integers there), subnormal rows and rows of one binade per value."""
import numpy as np
import pytest

from oracle import taq_oracle as O
from paper_2603_22943_amd import synth
from paper_2603_22943_amd import taq as T
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


def rows_of(kind, rows, cols, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    sig = rng.integers(1024, 2048, size=rows)
    if kind == "multiples":
        sig = 127 * rng.integers(9, 17, size=rows)
    amax = sig * 2.0 ** (-24 if kind == "subnormal" else -10)
    if kind == "subnormal":
        amax = rng.integers(1, 1024, size=rows) * 2.0 ** -24
    x = rng.uniform(-1, 1, size=(rows, cols)) * amax[:, None] * 2.0 ** -rng.integers(0, 12, size=(rows, cols))
    half = rng.random((rows, cols)) < 0.1
    x = np.where(half, np.sign(x) * amax[:, None] / 2, x).astype(np.float16)
    x = np.clip(x, -amax[:, None], amax[:, None]).astype(np.float16)
    x[np.arange(rows), rng.integers(0, cols, size=rows)] = amax * rng.choice((-1, 1), size=rows)
    return x


KINDS = ["any", "multiples", "subnormal"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("cols", [8, 1280, 2048])
def test_weight_rows(kind, cols):
    W = rows_of(kind, 301, cols, cols)
    code, scale = T.taq_quantize_weight(G.dev(W))
    want, s = O.quantize_weight(W)
    assert np.array_equal(code.cpu().numpy(), want) and np.array_equal(scale.cpu().numpy(), s.reshape(-1))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("C,H,N,w_layout", [(320, 8, 150, 1), (640, 8, 33, 0), (640, 10, 70, 1), (1280, 8, 19, 0), (1280, 20, 33, 1), (96, 4, 50, 0)])
def test_hidden_codes_and_the_block(kind, C, H, N, w_layout):
    L = synth.make_layer("rows", seed=C + N, B=2, N=N, C=C, H=H, Cc=64, T=77, bits_kv=8, trigger_positions=(3,), trigger_scale=3.0)
    hidden = rows_of(kind, 2 * N, C, C + N).reshape(2, N, C)
    g = G.GpuRun(L, hidden=hidden, w_layout=w_layout)
    want, scale = O.symq(hidden, 8)
    assert np.array_equal(g.taps["h_code"].reshape(want.shape), want)
    assert np.array_equal(g.taps["s_h"].reshape(-1), np.asarray(scale, dtype=np.float32).reshape(-1))
    quick = G.GpuRun(L, hidden=hidden, w_layout=w_layout, taps=False)
    assert np.array_equal(quick.out.view(np.uint16), g.out.view(np.uint16))
