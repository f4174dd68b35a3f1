"""The one-call token-sensitivity sweep where one text token takes almost the whole softmax row, or where a changed row takes
over a row that had none of it, against the oracle's sweep: rows in which the weight of the other tokens, or their distance from
the output, is far below the rounding of a number near 1."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import taq_oracle as O
from paper_2603_22943_amd import sensitivity, synth
from paper_2603_22943_amd import taq as T
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


def device_rows(L, bits, on):
    """K and V of every token as the library forms them, protected (on) or coded: float32 sums, in which now and then an fp16 rounding
    or the tie of a code falls to the other side than in the oracle's. One step of one channel meets scores of hundreds here, so both
    sides work on the same rows."""
    s = T.make_shape(B=L.B, N=1, C=L.C, H=L.H, T=L.T, Cc=L.Cc, bits_kv=bits, bits_q=16, bits_prob=16, bits_proj=16)
    mask = torch.full((L.B, L.T), on, dtype=torch.uint8, device=G.DEV)
    packed = T.taq_quantize_kv(G.dev(L.context), mask, G.dev(L.Wk), G.dev(L.Wv), bits, s)
    return {k: v.cpu().numpy() for k, v in T.taq_unpack_kv(packed, s).items()}


def oracle_sweep(L, bits, tokens, scale):
    full = device_rows(L, 16, 1)
    coded = {b: device_rows(L, b, 0) for b in bits}

    def block(mask, b):
        kv = O.quantize_kv(L.context, mask, L.Wk, L.Wv, b, L.H, bits_proj=16)
        on, new = kv.mask[:, :, None], {}
        for k in ("K16", "V16"):
            ref, got = getattr(kv, k), full[k].astype(np.float64)
            assert np.all(np.abs(got - ref)[kv.mask] <= 1.01 * np.spacing(np.abs(ref).astype(np.float16)).astype(np.float64)[kv.mask] + 1e-6)
            new[k] = np.where(on, got, 0.0)
        if b != 16:
            for k in ("k_code", "v_code"):
                ref, got = getattr(kv, k), np.where(on, 0, coded[b][k])
                assert np.abs(got - ref).max() <= 1 and np.count_nonzero(got != ref) <= 1 + 1e-3 * ref.size
                new[k] = got
            for k in ("s_K", "s_V"):
                ref, got = getattr(kv, k), np.where(kv.mask[:, None, :], 0, coded[b][k])
                assert np.allclose(got, ref, rtol=1e-5, atol=0)
                new[k] = got.astype(np.float32)
        kv = dataclasses.replace(kv, **new)
        return O.cross_attn(L.hidden, kv, None, None, None, None, L.bias_o, bits_q=16, bits_prob=16, bits_proj=16, Wq_f16=L.Wq,
                            Wo_f16=L.Wo, softmax_scale=scale).astype(np.float64)

    on = np.ones_like(L.mask)
    y = block(on, 16)
    out = {b: [] for b in bits}
    for b in bits:
        for i in tokens:
            m = on.copy()
            m[:, i] = 0
            out[b].append(np.mean((block(m, b) - y) ** 2))
    return y, {b: np.array(v) for b, v in out.items()}


@pytest.mark.parametrize("C,H,N,T_,factor,scale,outliers,bits", [
    (320, 8, 48, 12, 10.0, None, 0.0, (8, 4)),      # d = 40
    (640, 8, 33, 9, 10.0, None, 0.0, (8, 4)),       # d = 80
    (1280, 8, 32, 20, 10.0, None, 0.0, (8, 4)),     # d = 160
    (640, 8, 40, 17, 1.0, 1.0, 0.01, (8, 4)),
    (1280, 8, 20, 9, 1.0, 1.0, 0.01, (8, 4)),
    (320, 2, 40, 77, 30.0, None, 0.0, (8, 4)),
    (320, 8, 40, 12, 100.0, 1.0, 0.0, (8, 4)),      # scores hundreds apart: the other tokens underflow beside the largest
    (640, 20, 40, 5, 200.0, None, 0.0, (8, 4)),     # the 32-head specialisation
    (320, 8, 40, 1, 10.0, None, 0.0, (8, 4)),       # a single token keeps its weight of 1
    (320, 8, 40, 2, 100.0, None, 0.0, (8, 4)),
    (320, 4, 65, 96, 50.0, None, 0.0, (4,)),        # one width, the longest prompt
    (384, 12, 50, 33, 50.0, None, 0.0, (4,)),       # between the specialisations
    (640, 20, 1200, 12, 100.0, None, 0.0, (8, 4)),  # two passes over the rows
])
def test_sharp_rows(C, H, N, T_, factor, scale, outliers, bits):
    L = synth.make_layer("sharp", seed=C + H + N + T_, B=2, N=N, C=C, H=H, Cc=96, T=T_, bits_kv=8,
                         trigger_positions=(T_ // 2,), trigger_scale=3.0, outlier_frac=outliers, bias=True)
    L.hidden = (L.hidden.astype(np.float32) * factor).astype(np.float16)
    s = T.make_shape(B=2, N=N, C=C, H=H, T=T_, Cc=96, bits_q=16, bits_prob=16, bits_proj=16, softmax_scale=scale or 0.0)
    scales = torch.cat([torch.full((2 * C,), float("nan"), device=G.DEV), G.dev(L.bias_o)]).contiguous()
    tokens = list(range(T_))[-24:]
    got = sensitivity.token_sensitivity(G.dev(L.hidden), G.dev(L.context), G.dev(L.Wk), G.dev(L.Wv), G.dev(L.Wq), G.dev(L.Wo),
                                        scales, s, bits=bits, tokens=tokens)
    y, ref = oracle_sweep(L, bits, tokens, scale)
    n = y.size
    # Float32 scores of magnitude s carry an error of a few 2^-24 s, which the softmax turns into that relative error of the
    # weights (s up to 2000 here: 5e-4 of an entry's change, 1e-3 of its square). Beside that both sides round their
    # outputs to fp16, and one output in some hundred comes out one step apart: 2.2 / sqrt(n) bounds what that makes of a Delta of
    # half a step, a fiftieth of the mean squared step what it makes of a Delta of nothing.
    step = 0.02 * np.mean(np.spacing(np.abs(y).astype(np.float16)).astype(np.float64) ** 2)
    for b in bits:
        g, r = got[b].numpy(), ref[b]
        print(f"[sharp C={C} H={H} x{factor} scale={scale}] b={b}: max dev {np.max(np.abs(g - r) / (r + step)):.2e}, Delta {r.min():.2e} .. "
              f"{r.max():.2e}", flush=True)
        assert np.all(np.isfinite(g))
        assert np.all(np.abs(g - r) <= (2.2 / np.sqrt(n) + 2e-3) * r + step)
