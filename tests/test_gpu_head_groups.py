"""The head-group kernel of the C = 1280 and 640 layers: one and two tiles of 16 tokens per workgroup, the tail kernel or the stage path's last two
behind it, against the stage path, bit for bit. The waits that its image needs are checked on the generated code (CPU)."""
import numpy as np
import pytest
import torch

from paper_2603_22943_amd import taq as T


@pytest.mark.gpu
@pytest.mark.parametrize("B,N,H,more", [
    (1, 1, 8, dict()),
    (1, 33 * 16 - 15, 8, dict(w_layout=1)),               # two tiles per workgroup: the last group is half empty, its tile ragged
    (3, 201, 8, dict(prob_grid=1)),                       # an odd number of tiles per batch element
    (2, 509, 8, dict(w_layout=1, bits_kv=4, prob_grid=2)),  # ... with the stage path's kernels behind
    (4, 256, 8, dict(bits_kv=4)),
    (2, 16 * 48 - 7, 20, dict(w_layout=1)),               # heads of 64: 96 tiles
    (5, 317, 20, dict(w_layout=1, prob_grid=2)),
    (1, 16 * 60 - 1, 20, dict(w_layout=1, prob_grid=1)),  # one tile per workgroup, stage kernels behind
    (3, 33, 20, dict()),
    (1, 600, 8, dict(text=64)),                           # other lengths of text: one tile per workgroup
    (2, 330, 20, dict(text=96, w_layout=1)),
    (1, 16 * 96 - 3, 8, dict(w_layout=1)),                # one tile, stage kernels behind
    (12, 77, 8, dict()),                                  # ... 60 tiles that would be 36 workgroups of two
    (20, 80, 20, dict(w_layout=1, prob_grid=2)),
    (1, 16 * 64, 8, dict(text=48, w_layout=1)),
    # to_out: 2 or 4 output tiles per workgroup, K range shared by 4 or 2 wavefronts; 8; 10: the last size of each and the next
    (1, 16 * 6, 8, dict(w_layout=1)),
    (2, 16 * 3 - 5, 20, dict()),
    (1, 16 * 7, 20, dict(w_layout=1)),
    (3, 16 * 4 - 1, 8, dict(prob_grid=1)),
    (1, 16 * 13, 8, dict()),
    (1, 16 * 25, 20, dict()),
    (2, 16 * 13, 8, dict(w_layout=1)),
    (1, 16 * 32 - 9, 20, dict()),
])
@pytest.mark.parametrize("protected", [0, 3, 20])
def test_head_groups_and_stages_agree(B, N, H, more, protected):
    from test_gpu_token_tiles import Layer

    L = Layer(B, N, 1280, H, **more)
    L.mask.zero_()
    L.mask[:, 1 : 1 + 3 * protected : 3] = 1
    L.mask[:, : max(0, protected - int(L.mask[0].sum()))] = 1
    g = torch.Generator("cuda")
    g.manual_seed(protected)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    L.kv = T.taq_quantize_kv(normal(B, L.text, 64).half(), L.mask, (normal(1280, 64) * 0.1).half(), (normal(1280, 64) * 0.1).half(),
                             L.more["bits_kv"], L.shape(N))
    stages = L.run(tok_tile=32)
    assert np.array_equal(L.run(), stages)
    assert np.array_equal(L.run(tok_tile=16), stages)


@pytest.mark.gpu
@pytest.mark.parametrize("B,N,H,more,forced", [
    (1, 1, 8, dict(w_layout=1), 16),
    (1, 16 * 80 - 5, 8, dict(w_layout=1, prob_grid=1), 16),
    (4, 16 * 13, 8, dict(w_layout=1), 16),                  # to_out: 10 output tiles per workgroup
    (1, 16 * 64 - 1, 8, dict(), 16),
    (3, 201, 8, dict(bits_kv=4), 16),                       # row-major weights, one tile per workgroup
    (1, 1419, 8, dict(bits_kv=4), 16),                      # ... in more than one round
    (14, 77, 8, dict(), 16),
    (2, 1021, 8, dict(prob_grid=2), 16),
    (5, 33, 8, dict(text=64), 16),                          # other lengths of text
    (1, 1009, 8, dict(text=96, w_layout=1, prob_grid=2), 16),
    (1, 17, 10, dict(w_layout=1, prob_grid=2), 16),         # heads of 64
    (2, 16 * 51 - 9, 10, dict(w_layout=1), 16),
    (1, 810, 10, dict(bits_kv=4), 16),
    (3, 530, 10, dict(prob_grid=1), 16),                    # an odd number of tiles per batch element
    (2, 300, 10, dict(text=33), 16),
    (2, 300, 10, dict(text=96), 32),                        # more text than the single kernel has LDS for: against the stages
    (1, 16 * 102, 10, dict(text=81, w_layout=1, prob_grid=2), 32),
])
@pytest.mark.parametrize("protected", [0, 3, 20])
def test_head_groups_of_640_channels(B, N, H, more, forced, protected):
    """... and of the C = 640 layers of few tokens, against the single kernel, or the stages where there is none."""
    from test_gpu_token_tiles import Layer

    L = Layer(B, N, 640, H, **more)
    L.mask.zero_()
    L.mask[:, 1 : 1 + 3 * min(protected, 10) : 3] = 1
    L.mask[:, : max(0, protected - int(L.mask[0].sum()))] = 1
    g = torch.Generator("cuda")
    g.manual_seed(protected)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    L.kv = T.taq_quantize_kv(normal(B, L.text, 64).half(), L.mask, (normal(640, 64) * 0.1).half(), (normal(640, 64) * 0.1).half(),
                             L.more["bits_kv"], L.shape(N))
    assert np.array_equal(L.run(), L.run(tok_tile=forced))


@pytest.mark.gpu
@pytest.mark.parametrize("R,B,N,C,H,more", [
    (2, 1, 1, 1280, 8, dict(w_layout=1)),
    (3, 2, 23, 1280, 20, dict(w_layout=1)),                      # 12 tiles: one per workgroup
    (17, 1, 40, 1280, 8, dict(bits_kv=4)),                       # two, an odd number of them; a second launch of one request
    (17, 1, 16 * 103, 1280, 20, dict(w_layout=1)),               # ... of one that stages take
    (18, 1, 16 * 17 - 3, 320, 8, dict(w_layout=1)),              # the single kernel: 16, then two
    (5, 3, 70, 1280, 20, dict(prob_grid=1)),
    (2, 1, 16 * 100, 1280, 20, dict(w_layout=1, prob_grid=2)),   # the last size, and the next: request after request
    (2, 1, 16 * 101, 1280, 20, dict(w_layout=1)),
    (4, 1, 100, 1280, 8, dict(text=90)),
    (3, 1, 16 * 16, 640, 8, dict(w_layout=1)),                   # (and the next: the single kernel)
    (3, 1, 16 * 17, 640, 8, dict(w_layout=1)),
    (16, 2, 30, 640, 8, dict(bits_kv=4, prob_grid=1)),
    (5, 1, 150, 640, 10, dict(prob_grid=2)),
    (3, 2, 100, 640, 10, dict(text=96, w_layout=1)),
    (1, 1, 100, 640, 10, dict()),
])
def test_requests_of_one_launch(R, B, N, C, H, more):
    """Requests with weights, K~/V~ and hidden states of their own: grouped launches give the rows of single calls."""
    from test_gpu_token_tiles import Layer

    layers = []
    for r in range(R):
        L = Layer(B, N, C, H, **more)
        g = torch.Generator("cuda").manual_seed(100 + r)
        normal = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
        L.mask.zero_()
        L.mask[:, : (1, 0, 3, 20)[r % 4]] = 1
        L.kv = T.taq_quantize_kv(normal(B, L.text, 64).half(), L.mask, (normal(C, 64) * 0.1).half(), (normal(C, 64) * 0.1).half(), L.more["bits_kv"], L.shape(N))
        L.hidden = L.hidden.roll(3 * r, 1) * (1 + r)
        L.scales = L.scales * (1 + 0.25 * r)
        w = torch.randint(-127, 128, (C, C), generator=torch.Generator("cuda").manual_seed(r), device="cuda", dtype=torch.int8)
        L.w = T.taq_pack_weight(w, L.shape(N)) if more.get("w_layout") else w
        layers.append(L)
    s = layers[0].shape(N)
    reqs = [dict(hidden=L.hidden, qkv_packed=L.kv, Wq=L.w, Wo=L.w, scales=L.scales, trigger_mask=L.mask, out=torch.full_like(L.hidden, float("nan")))
            for L in layers]
    ws = torch.zeros(R * T.taq_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    for _ in range(2):  # (the second on what the first has left in the workspace)
        T.taq_cross_attn_batched(reqs, s, ws)
        for L, q in zip(layers, reqs):
            assert np.array_equal(q["out"].cpu().numpy().view(np.uint16), L.run(tok_tile=0))
            q["out"].fill_(float("nan"))


@pytest.mark.gpu
@pytest.mark.parametrize("B,N", [(160, 5), (69, 17)])
def test_chunks_of_tiles_give_the_same_rows(B, N):
    """Calls whose tiles do not all fit the static scratch: two chunks of 80 tiles, and of 69, the middle of the 35th batch element."""
    from test_gpu_token_tiles import Layer

    L = Layer(B, N, 1280, 20)
    whole = L.run(tok_tile=16)
    out = torch.full_like(L.hidden, float("nan"))
    T.taq_cross_attn_static(L.hidden, L.kv, L.w, L.w, L.scales, L.mask, L.shape(N, 16), out)
    assert np.array_equal(out.cpu().numpy().view(np.uint16), whole)


@pytest.mark.gpu
@pytest.mark.parametrize("R,B,N,C,H", [(1, 1, 5, 640, 8), (3, 1, 5, 640, 8), (1, 3, 33, 640, 10), (3, 3, 33, 640, 10), (1, 1, 16 * 72, 640, 8), (3, 1, 16 * 16, 640, 8),
                                       (1, 2, 77, 1280, 8), (3, 2, 77, 1280, 8), (1, 1, 16 * 60 - 1, 1280, 20), (3, 1, 16 * 60 - 1, 1280, 20)])
def test_nothing_is_written_past_the_workspace(R, B, N, C, H):
    """Calls that go through the workspace keep to taq_workspace_bytes() of their own shape, or R times as much."""
    from test_gpu_token_tiles import Layer

    L = Layer(B, N, C, H, w_layout=1)
    s, want = L.shape(N), L.run()
    n, past = R * T.taq_workspace_bytes(s), 1 << 16
    ws = torch.full((n + past,), 0xA5, dtype=torch.uint8, device="cuda")
    outs = [torch.full_like(L.hidden, float("nan")) for _ in range(R)]
    if R == 1:
        T.taq_cross_attn(L.hidden, L.kv, L.w, L.w, L.scales, L.mask, s, outs[0], ws[:n])
    else:
        T.taq_cross_attn_batched([dict(hidden=L.hidden, qkv_packed=L.kv, Wq=L.w, Wo=L.w, scales=L.scales, out=o) for o in outs], s, ws[:n])
    assert all(np.array_equal(o.cpu().numpy().view(np.uint16), want) for o in outs)
    assert bool((ws[n:] == 0xA5).all()) and not bool((ws[:n] == 0xA5).all())


@pytest.mark.parametrize("source", ["taq_heads160.hip", "taq_heads64.hip", "taq_heads80.hip", "taq_heads64x10.hip"])
def test_the_image_has_arrived(tmp_path, source):
    """Image and protected rows go straight into LDS for all wavefronts: a wavefront's own pieces have arrived at every barrier but the first
    (behind the codes of the hidden tile), and before its first exponential."""
    from test_image_waits import exponentials_with_lds_loads_in_flight
    from test_waits import assembly, barriers_with_lds_loads_in_flight

    bodies = {k: b for k, b in assembly(source, tmp_path).items() if "heads_kernel" in k}
    assert len(bodies) == (24 if source in ("taq_heads80.hip", "taq_heads64x10.hip") else 36)  # (C = 640: no two tiles per workgroup)
    for name, body in bodies.items():
        marked = [(no, "load_lds " + text if text.startswith("buffer_load") and text.endswith(" lds") else text, hand) for no, text, hand in body]
        barriers = [no for no, text, _ in body if text == "s_barrier"]
        assert sum(text.startswith("load_lds") for _, text, _ in marked) >= 2 and len(barriers) >= 6, name
        assert set(barriers_with_lds_loads_in_flight(marked)) <= {barriers[0]}, name
        assert not exponentials_with_lds_loads_in_flight(body), name
