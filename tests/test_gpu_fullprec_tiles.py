"""Tiles of the full-precision projections that the number of outputs selects. Every output is one chain of sums in K order, so a call
on many image tokens, which takes the large tiles, has the bits of calls on few of them."""
import numpy as np
import pytest
import torch

from paper_2603_22943_amd import taq as T

pytestmark = pytest.mark.gpu


def normal(seed, *shape, std=1.0):
    g = torch.Generator("cuda")
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * std).half()


def projections(B, N, C, H, text, Cc, bits_q, hidden):
    """Q~ codes' effect and all: the block with fp16 projections on `hidden` rows."""
    s = T.make_shape(B, hidden.shape[1], C, H, text, Cc, bits_q=bits_q, bits_proj=16)
    mask = torch.zeros((B, text), dtype=torch.uint8, device="cuda")
    mask[:, 1] = 1
    wk, wv, wq, wo = (normal(7 + i, C, k, std=k ** -0.5) for i, k in enumerate((Cc, Cc, C, C)))
    kv = T.taq_quantize_kv(normal(3, B, text, Cc), mask, wk, wv, 8, s)
    scales = torch.zeros(3 * C, device="cuda")
    return T.taq_cross_attn(hidden, kv, wq, wo, scales, mask, s).cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("B,N,C,H,bits_q", [
    (1, 1700, 640, 8, 8),   # 16 rows to a workgroup, a last one of four
    (2, 1041, 480, 10, 8),  # seven and a half chunks of K, columns that end within a tile
    (1, 3293, 320, 8, 8),
    (1, 1700, 672, 6, 4),   # ten and a half chunks of K
    (1, 8185, 640, 8, 8),   # 5120 workgroups of 16 rows: 32 rows to a workgroup, a last one of 25
    (2, 5121, 480, 10, 8),  # a last one of two
    (1, 7441, 672, 6, 4),   # of 17
    (1, 16369, 320, 8, 8),
])
def test_many_rows_have_the_bits_of_few(B, N, C, H, bits_q):
    hidden = normal(1, B, N, C)
    whole = projections(B, N, C, H, 9, 96, bits_q, hidden)
    for lo, hi in ((0, 1), (63, 130), (N - 37, N)):
        assert np.array_equal(whole[:, lo:hi], projections(B, N, C, H, 9, 96, bits_q, hidden[:, lo:hi].contiguous())), (lo, hi)


@pytest.mark.parametrize("C,H,n,times", [(640, 8, 33, 125), (1280, 8, 20, 90), (672, 6, 64, 50), (96, 4, 17, 1200)])
def test_sweep_over_repeated_rows(C, H, n, times):
    """Rows repeated leave every mean as it is, but for the order of its float64 sum (2^-53 a term, some thousand partial sums)."""
    Cc, text = 96, 5
    few = normal(2, 1, n, C)
    w = [normal(20 + i, C, k, std=k ** -0.5) for i, k in enumerate((Cc, Cc, C, C))]
    context, scales = normal(4, 1, text, Cc, std=2.0), torch.zeros(3 * C, device="cuda")

    def sweep(hidden):
        s = T.make_shape(1, hidden.shape[1], C, H, text, Cc, bits_q=16, bits_prob=16, bits_proj=16)
        return T.taq_token_sensitivity(hidden, context, *w, scales, range(text), (8, 4), s).cpu().numpy()

    a, b = sweep(few), sweep(few.repeat(1, times, 1))
    assert np.all(a[1] > 0) and np.all(np.abs(a - b) <= 1e-9 * a)


@pytest.mark.parametrize("C,H,n,times,text,bits,factor", [
    (96, 4, 17, 260, 17, (8, 4), 1.0),     # 1032 workgroups or more of one wavefront against few of four, two to six tiles of text
    (320, 8, 40, 52, 33, (4,), 1.0),
    (96, 4, 33, 130, 49, (8, 4), 1.0),
    (320, 8, 19, 112, 77, (8, 4), 1.0),
    (640, 8, 33, 64, 77, (4,), 1.0),
    (320, 2, 21, 400, 96, (8,), 1.0),
    (96, 4, 20, 210, 5, (4,), 1.0),        # one tile, one width
    (320, 4, 65, 66, 96, (8, 4), 50.0),    # rows that one token takes almost whole
    (96, 4, 31, 140, 33, (4,), 50.0),
])
def test_sweep_with_one_wavefront_has_the_bits_of_four(C, H, n, times, text, bits, factor):
    """As above, in the attention: one wavefront to 16 tokens and a head on the repeated rows, four on the few."""
    Cc = 96
    few = normal(2, 1, n, C) * factor
    w = [normal(20 + i, C, k, std=k ** -0.5) for i, k in enumerate((Cc, Cc, C, C))]
    context, scales = normal(4, 1, text, Cc, std=2.0), torch.zeros(3 * C, device="cuda")

    def sweep(hidden):
        s = T.make_shape(1, hidden.shape[1], C, H, text, Cc, bits_q=16, bits_prob=16, bits_proj=16)
        return T.taq_token_sensitivity(hidden, context, *w, scales, range(text), bits, s).cpu().numpy()

    assert (n + 31) // 32 * 2 * H <= 1024 < (n * times + 31) // 32 * 2 * H
    a, b = sweep(few), sweep(few.repeat(1, times, 1))
    assert a.max() > 0 and np.all(np.isfinite(a)) and np.all(np.abs(a - b) <= 1e-9 * a)
