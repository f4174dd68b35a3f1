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
        print(f"[sweep C={C} H={H} N={N}] b={b}: max dev {np.max(np.abs(g / ref[b] - 1)):.2e}, of the sum {abs(g.sum() / ref[b].sum() - 1):.2e}", flush=True)
        # Both sides round their outputs to fp16, and of n outputs about one in a hundred comes out one step apart (float32 against
        # float64 arithmetic in front of the rounding). With a change of s steps in the mean such a one is off by up to 2 / s of its
        # square: sqrt(0.01 n) * 2 / s of a sum of n, and 5 times that for the largest of a sweep; s is at least 0.45 at 8 bits
        # and, with steps of the grid 18 times as wide, 8 at 4 bits. The float32 factors themselves are good to 1e-3 of a square.
        assert np.all(np.abs(g / ref[b] - 1) <= (2.2 if b == 8 else 0.13) / np.sqrt(B * N * C) + 2e-3)
