"""The token sweep's product per head splits a float32 into three bfloat16 parts and an fp16 weight into two (csrc/taq_fp.hip,
gemm_nt_split_kernel): layers whose result hangs on the small parts, because the leading ones cancel, against float64. One text token, whose
V row is a column of Wv: the sweep's result is then the mean square of Wo (v' - v), v' its 4-bit row, beside a bias that takes Wo v away.

rows      pairs of channels with opposite weights and all but equal v' - v: one of 11 bits and one of 24 that begins with them
weights   pairs of channels with equal v' - v and weights that differ in their last three bits
"""
import numpy as np
import pytest
import torch

from paper_2603_22943_amd import taq as T

HEADS = [(4, 8), (4, 24), (8, 40), (4, 80), (2, 160)]  # heads of 8 to 160 channels, in steps of 32
AMAX = 71.0 * 64


def layer(kind, H, d):
    rng = np.random.default_rng(H + d)
    C, s = H * d, np.float32(AMAX) / np.float32(7)
    v = np.zeros(C, np.float16)
    for c in range(0, C, 2):
        if c % d == 0:
            v[c], v[c + 1] = AMAX, -AMAX  # (the grid of the head; no weight)
        elif kind == "rows":
            v[c] = s * np.float32(1 + rng.uniform(-0.06, 0.06))
            x = s - np.float32(v[c])
            t = np.float16(x)
            v[c + 1] = -(t if abs(np.float32(t)) <= abs(x) else np.nextafter(t, np.float16(0)))
        else:
            v[c] = v[c + 1] = s * np.float32(rng.integers(-6, 7) + rng.uniform(-0.4, 0.4))
    w = (rng.uniform(0.5, 1.0, (C, C // 2)) * rng.choice((-1, 1), (C, C // 2))).astype(np.float16)
    W = np.zeros((C, C), np.float16)
    if kind == "rows":
        W[:, 0::2], W[:, 1::2] = w, -w
    else:
        top, low = w.view(np.uint16) & 0xFFF8, rng.integers(0, 8, w.shape).astype(np.uint16)
        W[:, 0::2], W[:, 1::2] = (top | low).view(np.float16), -(top | (7 - low)).view(np.float16)
    W[:, [c for c in range(C) if c % d < 2]] = 0
    return C, v, W


def parts(x, n):
    out = []
    for _ in range(n):
        lead = (x.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
        out.append(lead.astype(np.float64))
        x = x - lead
    assert not x.any()
    return out


def expected(C, v, W, lost=None):
    v32, s = v.astype(np.float32), np.float32(AMAX) / np.float32(7)
    code = np.rint(v32 * np.float32(7) / np.float32(AMAX))
    change = code.astype(np.float32) * s - v32
    pv, pw = parts(change, 3), parts(W.astype(np.float32), 2)
    D = sum(pw[j] @ pv[i] for i in range(3) for j in range(2) if (i, j) != lost)
    return np.mean(D.astype(np.float16).astype(np.float64) ** 2)


@pytest.mark.parametrize("H,d", HEADS)
def test_every_product_counts(H, d):
    """Without any of them but the leading one, which cancels (any other sweep would show it), and the smallest (2^-24 of a product) the
    expectation is off by more than the GPU's test allows. On the CPU."""
    for lost in ((1, 0), (2, 0), (0, 1), (1, 1)):
        off = [abs(expected(*layer(kind, H, d), lost=lost) / expected(*layer(kind, H, d)) - 1) for kind in ("rows", "weights")]
        assert max(off) > 3e-3, (lost, off)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["rows", "weights"])
@pytest.mark.parametrize("H,d", HEADS)
def test_sweep_of_one_token(kind, H, d):
    C, v, W = layer(kind, H, d)
    N, Cc = 33, 32
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    context = np.zeros((1, 1, Cc), np.float16)
    context[0, 0, 0] = 1
    Wv = np.zeros((C, Cc), np.float16)
    Wv[:, 0] = v
    bias = -(W.astype(np.float64) @ v.astype(np.float64)).astype(np.float32)
    scales = torch.cat([torch.zeros(2 * C, device="cuda"), dev(bias)])
    hidden = np.random.default_rng(1).normal(size=(1, N, C)).astype(np.float16)
    s = T.make_shape(1, N, C, H, 1, Cc, bits_q=16, bits_prob=16, bits_proj=16)
    got = T.taq_token_sensitivity(dev(hidden), dev(context), dev(Wv), dev(Wv), dev(W), dev(W), scales, range(1), (4,), s).cpu().numpy().reshape(-1)[0]
    # float32 sums of C products x w: C 2^-24 of their magnitudes, 1e-3 of an output here at most and of either sign in C of them; fp16 outputs: 2^-12
    # of each, of either sign. (Where Wo v is taken away, what is left of it stands in both outputs.)
    want = expected(C, v, W)
    print(f"[split {kind} H={H} d={d}] {got / want - 1:+.1e}", flush=True)
    assert abs(got / want - 1) <= 1e-3
