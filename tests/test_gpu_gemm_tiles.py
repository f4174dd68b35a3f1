"""Tiles of to_q and to_out that the number of workgroups selects, and odd numbers of K steps, whose first step stands by itself. The
rows of a call that takes the tile named are, bit for bit, those of calls on a few tokens, which take the smallest tiles."""
import numpy as np
import pytest

from test_gpu_token_tiles import Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,C,H", [
    (2, 1023, 1280, 20),  # to_q 96 x 128, two wavefronts a head; to_out 128 x 80
    (8, 383, 1280, 8),    # to_q 96 x 160; to_out 128 x 128
    (3, 2049, 1280, 8),   # to_q 128 x 160, two wavefronts a head
    (2, 200, 64, 4),      # one K step
    (1, 1100, 960, 12),   # 15 K steps, heads of 80
    (1, 1537, 320, 2),    # 5 K steps, heads of 160
    (3, 1200, 320, 20),   # 5 K steps, heads of 16: a block each
    (2, 700, 672, 6),     # 10 and a half K steps, heads of 112
])
@pytest.mark.parametrize("w_layout", [0, 1])
def test_tiles_do_not_change_results(B, N, C, H, w_layout):
    if w_layout and C % 64:
        pytest.skip("no operand-ordered copy of such a matrix")
    L = Layer(B, N, C, H, w_layout=w_layout)
    whole = L.run()
    for lo, hi in ((0, 1), (95, 130), (N - 37, N)):
        assert np.array_equal(whole[:, lo:hi], L.run(lo, hi)), (lo, hi)


@pytest.mark.parametrize("B,N,H,w_layout", [(1, 816, 20, 1), (1, 817, 20, 1), (1, 817, 20, 0), (1, 512, 8, 0), (1, 513, 8, 0), (1, 1025, 8, 1)])
def test_head_groups_and_stages_agree_where_the_rule_changes(B, N, H, w_layout):
    L = Layer(B, N, 1280, H, w_layout=w_layout)
    assert np.array_equal(L.run(), L.run(tok_tile=16))
