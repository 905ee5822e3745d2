"""Layers of one topk_attn_decode_layers call share their launches: every output is bit for bit that of a call per layer
(which the other tests judge against the oracle), whatever path the layers take and however many of them join."""
import numpy as np
import pytest
import torch

from paper_2502_06766_amd import topk_attn as ta
from paper_2502_06766_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda"
TORCH = {wl.F32: torch.float32, wl.F16: torch.float16, wl.BF16: torch.bfloat16}

# layers, sequences, (query, KV) heads, d, dtype, tokens per layer (cycled), k per layer (cycled), window, forced redo, key rows repeated
CASES = {
    "lists_8x48k_all_shares_in_one_workgroup": (8, 1, 32, 8, 128, wl.F16, (48001,), (512, 600, 700, 1000), 0, 0, 0),
    "lists_7_layers_two_shares_a_workgroup": (7, 1, 16, 4, 64, wl.BF16, (33000, 32999), (300, 411), 0, 0, 0),
    "lists_ragged_window": (4, 2, 8, 2, 128, wl.F16, (70000, 20001, 60000), (64, 700), 256, 0, 0),
    "lists_more_rows_than_are_asked_for_at_once": (8, 1, 32, 8, 128, wl.F16, (33001,), (2000, 1025, 1024, 2047), 0, 0, 0),
    "lists_more_rows_than_shares": (8, 1, 32, 8, 64, wl.BF16, (33001,), (3, 5, 9, 1), 0, 0, 0),
    "lists_row_tiles": (2, 1, 16, 2, 128, wl.BF16, (40003,), (500, 333), 100, 0, 0),
    "lists_redo": (4, 1, 8, 2, 64, wl.F16, (40000,), (256,), 0, 1, 0),
    "lists_tied": (4, 1, 8, 2, 64, wl.F16, (40000,), (256, 300), 0, 0, 40),
    "lists_then_rows": (4, 1, 8, 2, 128, wl.BF16, (40000, 40000, 9000, 9000), (256, 300), 0, 0, 0),
    "rows": (8, 1, 32, 8, 64, wl.BF16, (4096, 4001, 3000), (64, 65, 200), 0, 0, 0),
    "rows_window_many_heads": (4, 10, 32, 8, 64, wl.F16, (2040, 2000), (64, 33), 64, 0, 0),
    "rows_f32": (3, 1, 4, 1, 64, wl.F32, (5000, 7001), (100, 40), 0, 0, 0),
    "short": (4, 6, 8, 4, 64, wl.F16, (500, 77), (30, 90), 0, 0, 0),
    "few_tokens": (2, 1, 2, 1, 32, wl.F16, (1, 70), (5, 100), 0, 0, 0),
    "tail_each_on_its_own": (2, 1, 8, 2, 64, wl.F16, (70000,), (5000,), 0, 0, 0),
}


@pytest.mark.parametrize("name", CASES)
def test_layers_in_one_call_equal_a_call_per_layer(name):
    L, B, Hq, Hkv, d, dtype, tokens, ks, window, redo, repeat = CASES[name]
    ks = [ks[l % len(ks)] for l in range(L)]
    cache = ta.TopkAttnCache(L, B, Hq, Hkv, d, max(tokens), max(ks), dtype, max_window=window)
    try:
        g = torch.Generator(device=DEV)
        g.manual_seed(1)
        for l in range(L):
            for b in range(B):
                n = max(1, tokens[l % len(tokens)] - 37 * b)
                K, V = (torch.randn((Hkv, n, d), generator=g, device=DEV).to(TORCH[dtype]) for _ in range(2))
                if repeat:                                     # most keys are copies of a few: long lists, ties
                    K[:, :n * 9 // 10] = K[:, torch.arange(n * 9 // 10, device=DEV) % repeat]
                cache.append(l, b, K, V, head_major=True)
        q = torch.randn((L, B, Hq, d), generator=g, device=DEV).to(TORCH[dtype])
        if redo:
            ta.topk_attn_debug_force_redo(cache.h, redo)
        single = [cache.decode(l, q[l], ks[l], window=window) for l in range(L)]
        records = ta.topk_attn_last_selection_records(cache.h, B * Hq) if name.startswith("lists_8") else None
        fallbacks = ta.topk_attn_last_fallbacks(cache.h)
        st = torch.cuda.current_stream().cuda_stream
        for want in (True, False):                             # with the selection, and without (kept in the workspace)
            out = torch.full((L, B, Hq, d), 7.0, device=DEV)
            lse = torch.full((L, B, Hq), 7.0, device=DEV)
            idx = torch.full((B * Hq * sum(ks),), -7, dtype=torch.int32, device=DEV)
            vals = torch.full((B * Hq * sum(ks),), 7.0, device=DEV)
            ta.topk_attn_decode_layers(cache.h, 0, ks, q.data_ptr(), window, out.data_ptr(), idx.data_ptr() if want else 0,
                                       vals.data_ptr() if want else 0, lse.data_ptr(), st)
            torch.cuda.synchronize()
            at = 0
            for l in range(L):
                n = B * Hq * ks[l]
                assert torch.equal(out[l], single[l][0]) and torch.equal(lse[l], single[l][3]), f"layer {l}"
                if want:
                    assert torch.equal(idx[at:at + n], single[l][1].flatten()), f"layer {l}"
                    assert torch.equal(vals[at:at + n], single[l][2].flatten()), f"layer {l}"
                at += n
            assert ta.topk_attn_last_fallbacks(cache.h) == fallbacks
            if records is not None:
                assert ta.topk_attn_last_selection_records(cache.h, B * Hq) == records
    finally:
        cache.close()


@pytest.mark.parametrize("tokens,k", [(30000, 300), (5000, 64)])
def test_layers_over_a_smaller_workspace(tokens, k):
    """A workspace with room for one layer, two, or all (and a few bytes short of that) gives the same bits."""
    L, Hq, Hkv, d = 8, 8, 2, 64
    cfg = ta.make_config(L, 1, Hq, Hkv, d, tokens, k, ta.F16)
    sizes = [ta.topk_attn_layers_workspace_bytes(cfg, n) for n in (1, 2, 8)]
    assert sizes[0] == ta.topk_attn_workspace_bytes(cfg) < sizes[1] < sizes[2] == ta.topk_attn_layers_workspace_bytes(cfg)
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    K, V = (torch.randn((L, Hkv, tokens, d), generator=g, device=DEV).half() for _ in range(2))
    q = torch.randn((L, 1, Hq, d), generator=g, device=DEV).half()
    kv = torch.empty(ta.topk_attn_kv_bytes(cfg), dtype=torch.uint8, device=DEV)
    cfg.kv_storage, cfg.kv_bytes = kv.data_ptr(), kv.numel()
    st = torch.cuda.current_stream().cuda_stream
    results = []
    for size in [*sizes, sizes[2] - 256]:
        ws = torch.full((size + 256,), 0xEE, dtype=torch.uint8, device=DEV)
        cfg.workspace, cfg.workspace_bytes = ws.data_ptr(), size
        h = ta.topk_attn_create(cfg)
        try:
            for l in range(L):
                ta.topk_attn_append_kv(h, l, 0, K[l].data_ptr(), V[l].data_ptr(), tokens, d, tokens * d, st)
            out = torch.empty((L, 1, Hq, d), device=DEV)
            idx = torch.empty((L, 1, Hq, k), dtype=torch.int32, device=DEV)
            ta.topk_attn_decode_layers(h, 0, [k] * L, q.data_ptr(), 0, out.data_ptr(), idx.data_ptr(), stream=st)
            torch.cuda.synchronize()
            assert (ws[size:] == 0xEE).all()
            results.append((out, idx))
        finally:
            ta.topk_attn_destroy(h)
    for out, idx in results[1:]:
        assert torch.equal(out, results[0][0]) and torch.equal(idx, results[0][1])
    cfg.workspace_bytes = sizes[0] - 1
    with pytest.raises(ta.TopkAttnError) as e:
        ta.topk_attn_create(cfg)
    assert e.value.code == ta.ENOMEM


@pytest.mark.parametrize("L,Hq,Hkv,d,ks", [
    (4, 32, 8, 128, (700, 701, 300, 1000)),          # workgroups that take two shares of eight, so some do not hold the first row
    (2, 32, 8, 64, (256, 900)),
    (8, 32, 8, 256, (3, 200)),                       # one workgroup a head; shares without a row
])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_value_rows_that_were_not_selected_are_not_read(L, Hq, Hkv, d, ks, bad):
    """Every value row that no head of its KV head selected is Inf or NaN: outputs stay finite and equal a call per layer."""
    N, ks = 30001, [ks[l % len(ks)] for l in range(L)]
    cache = ta.TopkAttnCache(L, 1, Hq, Hkv, d, N, max(ks), wl.F16)
    try:
        g = torch.Generator(device=DEV)
        g.manual_seed(3)
        K, V = (torch.randn((L, Hkv, N, d), generator=g, device=DEV).half() for _ in range(2))
        q = torch.randn((L, 1, Hq, d), generator=g, device=DEV).half()
        for l in range(L):
            cache.append(l, 0, K[l], V[l], head_major=True)
            sel = cache.decode(l, q[l], ks[l])[1].view(Hkv, -1).long()
            keep = torch.zeros((Hkv, N), dtype=torch.bool, device=DEV).scatter_(1, sel, True)
            cache.reset(l, 0)
            cache.append(l, 0, K[l], torch.where(keep[..., None], V[l], torch.full_like(V[l], bad)), head_major=True)
        single = torch.stack([cache.decode(l, q[l], ks[l])[0] for l in range(L)])
        assert torch.isfinite(single).all()
        for _ in range(3):
            out = torch.empty((L, 1, Hq, d), device=DEV)
            ta.topk_attn_decode_layers(cache.h, 0, ks, q.data_ptr(), 0, out.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert torch.equal(out, single)
    finally:
        cache.close()


def test_workspace_arrays_after_a_joined_call():
    """What a joined call leaves for its last layer is what that layer leaves alone."""
    L, Hq, Hkv, d, N, k = 4, 8, 2, 64, 30000, 300
    cache = ta.TopkAttnCache(L, 1, Hq, Hkv, d, N, k, wl.F16)
    try:
        g = torch.Generator(device=DEV)
        g.manual_seed(5)
        for l in range(L):
            K, V = (torch.randn((Hkv, N, d), generator=g, device=DEV).half() for _ in range(2))
            cache.append(l, 0, K, V, head_major=True)
        q = torch.randn((L, 1, Hq, d), generator=g, device=DEV).half()
        out = torch.empty((L, 1, Hq, d), device=DEV)

        def arrays():
            torch.cuda.synchronize()
            n_seg = ta.topk_attn_debug_read_workspace_dims(cache.h)[4]
            assert 0 < n_seg < 1024
            read = {n: ta.topk_attn_debug_read_workspace(cache.h, n, np.uint32, n_seg * Hq) for n in ("seg_cnt", "seg_max")}
            read["thr"] = ta.topk_attn_debug_read_workspace(cache.h, "thr", np.uint32, Hq)
            return read, ta.topk_attn_last_selection_records(cache.h, Hq)

        cache.decode(L - 1, q[L - 1], k)
        alone = arrays()
        ta.topk_attn_decode_layers(cache.h, 0, [k] * L, q.data_ptr(), 0, out.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
        joined = arrays()
        assert joined[1] == alone[1]
        for name in alone[0]:
            assert (joined[0][name] == alone[0][name]).all(), name
    finally:
        cache.close()


def test_layers_in_one_call_under_graph_capture():
    """Replays with changing queries, with eager work in between, equal the eager results."""
    L, Hq, Hkv, d, N, ks = 4, 8, 2, 64, 30000, [200, 220, 240, 260]
    cache = ta.TopkAttnCache(L, 1, Hq, Hkv, d, N, max(ks), wl.F16)
    try:
        g = torch.Generator(device=DEV)
        g.manual_seed(2)
        for l in range(L):
            K, V = (torch.randn((Hkv, N, d), generator=g, device=DEV).half() for _ in range(2))
            cache.append(l, 0, K, V, head_major=True)
        q = torch.randn((L, 1, Hq, d), generator=g, device=DEV).half()
        out = torch.empty((L, 1, Hq, d), device=DEV)

        def call():
            ta.topk_attn_decode_layers(cache.h, 0, ks, q.data_ptr(), 0, out.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)

        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        for i in range(4):
            q.copy_(torch.randn((L, 1, Hq, d), generator=g, device=DEV).half())
            graph.replay()
            torch.cuda.synchronize()
            got = out.clone()
            want = torch.stack([cache.decode(l, q[l], ks[l])[0] for l in range(L)])
            torch.cuda.synchronize()
            assert torch.equal(got, want), i
    finally:
        cache.close()
