"""Protected rows as the attention kernels fetch them: the lanes of slots past the last one take no part in the loads. Counts around
the four slots of a lane and the sixteen of a tile, per batch element different, in every kernel family (qkv_packed starts as NaN
patterns, so that a slot nobody wrote shows up)."""
import numpy as np
import pytest

from paper_2603_22943_amd import synth
from tests import gpu_helpers as G
from tests.test_gpu_parity import check_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H", [(320, 8), (640, 8), (640, 10), (1280, 8), (1280, 20), (320, 2), (960, 12), (480, 12), (96, 6)])
@pytest.mark.parametrize("counts", [(0, 1, 4), (5, 15, 16), (17, 33, 3)])
def test_slots_past_the_last_are_not_read(C, H, counts):
    L = synth.make_layer("few", seed=C + H + counts[0], B=3, N=21, C=C, H=H, Cc=64, T=77, bits_kv=8, trigger_scale=3.0)
    rng = np.random.Generator(np.random.PCG64(C + counts[1]))
    for b, n in enumerate(counts):
        L.mask[b, rng.choice(77, size=n, replace=False)] = 1
    check_layer(L, f"slots C={C} H={H} ntrig={counts}")
    taps = G.GpuRun(L)  # (the builds with a fixed number of text tiles, and both ways through the C = 1280 layers)
    for tok_tile in (0, 16, 32) if C == 1280 else (0,):
        assert np.array_equal(G.GpuRun(L, taps=False, tok_tile=tok_tile).out.view(np.uint16), taps.out.view(np.uint16))


@pytest.mark.parametrize("counts", [(0, 1, 4), (5, 15, 16), (17, 33, 3)])
def test_slots_past_the_last_have_no_weight_on_the_log2_grid(counts):
    """Ten heads, run-time length of text: minus infinity by selects (csrc/taq_fused_kernel.h, SELECT)."""
    L = synth.make_layer("few", seed=7 + counts[0], B=3, N=21, C=640, H=10, Cc=64, T=40, bits_kv=8, trigger_scale=3.0)
    rng = np.random.Generator(np.random.PCG64(counts[1]))
    for b, n in enumerate(counts):
        L.mask[b, rng.choice(40, size=n, replace=False)] = 1
    check_layer(L, f"slots log2 ntrig={counts}", prob_grid="log2")


@pytest.mark.parametrize("protected", [0, 3, 16, 19])
def test_slots_past_the_last_with_64_tokens_to_a_workgroup(protected):
    """Four token tiles, operand-ordered weights: the same."""
    L = synth.make_layer("few", seed=protected, B=2, N=8185, C=640, H=8, Cc=64, T=77, bits_kv=8, trigger_scale=3.0)
    L.mask[:] = 0
    L.mask[:, 5:5 + protected] = 1
    wide = G.GpuRun(L, taps=False, w_layout=1)
    assert np.array_equal(wide.out.view(np.uint16), G.GpuRun(L, taps=False, w_layout=1, tok_tile=16).out.view(np.uint16))
