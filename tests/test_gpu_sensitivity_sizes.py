"""The one-call token-sensitivity sweep at the edges of its kernels' ranges, against the oracle's sweep: ragged image-token
counts, head counts on both sides of each specialisation, head dimensions that end in half a K step, the longest prompt,
channel counts that are no multiple of 64, several passes over the rows, one width, a subset with a repeated token."""
import numpy as np
import pytest
import torch

from paper_2603_22943_amd import sensitivity, synth
from paper_2603_22943_amd import taq as T
from tests import gpu_helpers as G
from tests.test_gpu_sensitivity import oracle_sweep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H,B,N,T_,bits,tokens", [
    (96, 4, 2, 33, 16, (8, 4), None),
    (64, 8, 1, 1, 17, (4,), None),          # d = 8: half a step of 16
    (320, 8, 1, 31, 5, (4, 8), [4, 0, 4]),
    (320, 2, 1, 20, 6, (8, 4), None),       # d = 160
    (96, 12, 3, 40, 4, (8, 4), None),       # between the specialisations
    (640, 20, 1, 70, 5, (4,), [1, 3]),
    (96, 4, 1, 65, 96, (8,), [0, 15, 16, 95]),
])
def test_sweep_sizes(C, H, B, N, T_, bits, tokens):
    L = synth.make_layer("sweep", seed=C + H + N, B=B, N=N, C=C, H=H, Cc=96, T=T_, bits_kv=8, trigger_positions=(1,),
                         trigger_scale=3.0, bias=True)
    s = T.make_shape(B=B, N=N, C=C, H=H, T=T_, Cc=96, bits_q=16, bits_prob=16, bits_proj=16)
    scales = torch.cat([torch.full((2 * C,), float("nan"), device=G.DEV), G.dev(L.bias_o)]).contiguous()
    got = sensitivity.token_sensitivity(G.dev(L.hidden), G.dev(L.context), G.dev(L.Wk), G.dev(L.Wv), G.dev(L.Wq), G.dev(L.Wo),
                                        scales, s, bits=bits, tokens=tokens)
    toks = list(range(T_)) if tokens is None else tokens
    ref = oracle_sweep(L, bits, toks, True)
    for b in bits:
        g = got[b].numpy()
        assert g.shape == (len(toks),)
        # at 8 bits Delta is a few fp16 steps of few outputs here; the sum over the sweep averages over them
        print(f"[sweep C={C} H={H} N={N}] b={b}: max dev {np.max(np.abs(g / ref[b] - 1)):.2e}, of the sum {abs(g.sum() / ref[b].sum() - 1):.2e}", flush=True)
        assert np.all(np.abs(g / ref[b] - 1) <= (0.5 if b == 8 else 0.1) / np.sqrt(max(1.0, B * N * C / 2048)) + 1e-2)
