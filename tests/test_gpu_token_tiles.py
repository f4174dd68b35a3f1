"""Kernels chosen by the number of image tokens: 48 and 64 tokens per workgroup where that saves rounds of workgroups, and the
block sizes of the kernel-per-stage path. Every choice gives the bits of the 16-token kernels, or of its own small blocks."""
import numpy as np
import pytest
import torch

from paper_2603_22943_amd import taq as T

pytestmark = pytest.mark.gpu


class Layer:
    def __init__(self, B, N, C, H, text=77, bits_kv=8, w_layout=0, prob_grid=0):
        g = torch.Generator("cuda")
        g.manual_seed(B + N + C + H)
        normal = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
        self.B, self.N, self.C, self.H, self.text = B, N, C, H, text
        self.more = dict(bits_kv=bits_kv, w_layout=w_layout, prob_grid=prob_grid)
        self.mask = torch.zeros((B, text), dtype=torch.uint8, device="cuda")
        self.mask[:, text // 2] = 1
        s = self.shape(N)
        code, scale = T.taq_quantize_weight((normal(C, C) * C ** -0.5).half())
        self.w = T.taq_pack_weight(code, s) if w_layout else code
        self.scales = torch.cat([scale, scale, normal(C)])
        wk, wv = (normal(C, 64) * 0.1).half(), (normal(C, 64) * 0.1).half()
        self.kv = T.taq_quantize_kv(normal(B, text, 64).half(), self.mask, wk, wv, bits_kv, s)
        self.hidden = normal(B, N, C).half()

    def shape(self, N, tok_tile=0):
        return T.make_shape(self.B, N, self.C, self.H, self.text, 64, tok_tile=tok_tile, **self.more)

    def run(self, lo=0, hi=None, tok_tile=0):
        hidden = self.hidden[:, lo:hi].contiguous()
        s = self.shape(hidden.shape[1], tok_tile)
        out = torch.full_like(hidden, float("nan"))
        ws = torch.zeros(T.taq_workspace_bytes(s), dtype=torch.uint8, device="cuda")
        T.taq_cross_attn(hidden, self.kv, self.w, self.w, self.scales, self.mask, s, out, ws)
        return out.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("B,N,H,more", [
    (1, 8193, 8, dict(w_layout=1)),                            # one tile more than a round of 32 tokens
    (2, 6131, 8, dict(bits_kv=4)),                             # 48 tokens, ragged, row-major
    (3, 5400, 8, dict(prob_grid=2, w_layout=1)),               # 64 tokens, a last tile of 24
    (2, 8185, 8, dict(bits_kv=4, prob_grid=1)),                # 64 tokens, row-major
    (1, 11003, 10, dict(prob_grid=2)),
    (2, 6144, 10, dict(bits_kv=4, w_layout=1)),
])
def test_larger_token_tiles_give_the_same_bits(B, N, H, more):
    L = Layer(B, N, 640, H, **more)
    assert np.array_equal(L.run(), L.run(tok_tile=16))


@pytest.mark.parametrize("C,H", [(96, 12), (128, 4), (480, 10), (512, 8), (320, 4), (576, 6), (448, 4), (640, 5), (864, 6), (320, 2), (768, 12)])
@pytest.mark.parametrize("w_layout", [0, 1])
def test_stage_path_blocks_do_not_change_results(C, H, w_layout):
    """Heads of one to ten 16-channel blocks; text on both sides of 65 to 80 tokens. The large blocks (all tokens in one call) and
    the small ones (a few tokens per call, with a ragged last tile) give the same rows."""
    if w_layout and C % 64:
        pytest.skip("no operand-ordered copy of such a matrix")
    N = 3 * 2 ** 20 // ((C // H + 15) // 16 * 16 * H) + 5  # more small blocks than the rule for them allows
    for text in (64, 77, 81):
        L = Layer(2, N, C, H, text=text, w_layout=w_layout)
        whole = L.run()
        for lo, hi in ((0, 1), (16, 33), (N - 85, N)):
            assert np.array_equal(whole[:, lo:hi], L.run(lo, hi)), (text, lo, hi)
