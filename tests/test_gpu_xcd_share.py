"""The stage path's kernels deal their work to the XCDs in eighths of its items: numbers of token tiles and of workgroups that do not
divide by 8, fewer than 8 of them, and a call that goes through its tiles in chunks. The rows are, bit for bit, those of other splits."""
import numpy as np
import pytest
import torch

from paper_2603_22943_amd import taq as T
from test_gpu_token_tiles import Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,C,H", [
    (2, 784, 1280, 20),   # to_q, to_out: 25 blocks of 20 workgroups
    (1, 1088, 768, 12),   # attention: 17 groups of 12 heads
    (3, 1601, 512, 8),    # a group of the attention per batch element that is mostly empty
    (2, 11003, 320, 4),   # two token tiles per wavefront, heads of 80
    (5, 37, 96, 4),       # a few workgroups
    (7, 1, 64, 1),        # one tile per batch element, one head
])
def test_rows_do_not_depend_on_the_split(B, N, C, H):
    L = Layer(B, N, C, H)
    whole = L.run(tok_tile=32)
    for lo, hi in ((0, 1), (N // 3, N // 3 + min(N, 40)), (max(N - 23, 0), N)):
        assert np.array_equal(whole[:, lo:hi], L.run(lo, hi, tok_tile=32)), (lo, hi)


@pytest.mark.parametrize("B,N", [(160, 5), (69, 17)])
def test_chunks_of_tiles_give_the_same_rows(B, N):
    """All tiles of these calls take 20.1 and 17.3 MB, the static scratch has 16.8: two chunks of 80 tiles, and of 69, the middle of the
    35th batch element."""
    L = Layer(B, N, 1280, 20)
    s = L.shape(N, 32)
    whole = L.run(tok_tile=32)
    out = torch.full_like(L.hidden, float("nan"))
    T.taq_cross_attn_static(L.hidden, L.kv, L.w, L.w, L.scales, L.mask, s, out)
    assert np.array_equal(out.cpu().numpy().view(np.uint16), whole)
