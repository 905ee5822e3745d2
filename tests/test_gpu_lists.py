"""Candidate lists the one-launch selection (csrc/attend.hip) cannot take as they are: longer than a workgroup's registers, or with
a segment that overflowed.  Groups of identical keys make them (a quarter of the cache that scores alike, just below the k-th
score, is a list of tens of thousands).  All elements of q and K are small multiples of a power of two, so the
scores are exact in fp32 and the selection has to equal the oracle's, ties to the lower position."""
import numpy as np
import pytest
import torch

import helpers as H
from oracle import c_oracle
from paper_2502_06766_amd import topk_attn as ta
from paper_2502_06766_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0) if torch.cuda.is_available() else None
IN_REGISTERS = 10240            # candidates a workgroup takes


def make_tied(seed, M, Hq, Hkv, N, d, groups, hot=None):
    """q [M, Hq, d], K, V [Hkv, N, d] (float32, exact in 16 bits).  groups: (share of the cache, score in standard deviations);
    hot: positions of one more group, four standard deviations up.  The queries of a chunk differ in one channel, so that a
    group scores alike for all of them."""
    g = np.random.default_rng(seed)
    q = np.repeat(g.integers(-3, 4, (1, Hq, d)).astype(np.float32) / 16, M, axis=0)
    for m in range(1, M):
        q[m, :, m % d] += 1 / 16
    K = g.integers(-8, 9, (Hkv, N, d)).astype(np.float32)
    V = g.standard_normal((Hkv, N, d)).astype(np.float32)
    sigma = np.sqrt((17.0 ** 2 - 1) / 12)
    for h in range(Hkv):
        Q = q[0, h * (Hq // Hkv):(h + 1) * (Hq // Hkv)].astype(np.float64)
        at = lambda z: np.rint(8 * np.linalg.lstsq(Q, z * sigma * np.linalg.norm(Q, axis=1), rcond=None)[0]) / 8
        perm = g.permutation(N)
        for share, z in groups:
            n = int(share * N)
            K[h, perm[:n]] = at(z)
            perm = perm[n:]
        if hot is not None:
            K[h, hot] = at(4.0)
    return q, K, V


def check_exact(res, q, K, V, dtype, k, causal, window, label):
    """res: (out, idx, vals, lse) of one sequence, numpy, [M, Hq, ...]."""
    M, Hq, _ = q.shape
    N = K.shape[1]
    vmax = float(np.abs(wl.widen(V, dtype)).max())
    for m in range(M):
        n = N - (M - 1 - m) if causal else N
        Km, Vm = (K, V) if n == N else (np.ascontiguousarray(K[:, :n]), np.ascontiguousarray(V[:, :n]))
        ref = c_oracle.topk_attention_window(q[m], Km, Vm, dtype, k, window)
        H.check_against_oracle(*(r[m] for r in res), ref, np.full(Hq, 1e-30), min(k, n - window), H.out_tolerance(dtype), vmax,
                               f"{label} query {m}")


def how_selected(cache, rows):
    """Per row: what became of its list, from the records and the scan's counts."""
    rec = ta.topk_attn_last_selection_records(cache.h, rows)
    dims = ta.topk_attn_debug_read_workspace_dims(cache.h)
    n_seg, seg_cap, bnd_cap = dims[4], dims[5], dims[1]
    cnt = ta.topk_attn_debug_read_workspace(cache.h, "seg_cnt", np.uint32, n_seg * rows).reshape(rows, n_seg)
    res, fallbacks = [], 0
    for r, c in zip(rec, cnt):
        over, cut = bool(c.max() > seg_cap), r[1] + r[3]
        if r[0] & 0xFF == 1:
            res.append("row")
        elif not over and c.sum() <= IN_REGISTERS:
            res.append("short")
        else:
            res.append(("rescored" if over else "long") + (", tied" if cut > IN_REGISTERS else ""))
        fallbacks += over or r[0] & 0xFF == 1 or r[3] > bnd_cap
    return res, fallbacks


@pytest.mark.parametrize("expect,dtype,M,Hq,Hkv,N,d,k,window,groups", [
    ("long", wl.F16, 1, 4, 2, 131072, 64, 2048, 0, [(0.25, 1.9)]),              # eight workgroups per head
    # one workgroup per head, causal chunk, window.  (The threshold is the 33rd of 1024 samples.  1.6 % of the keys, 16 +- 4 of the samples,
    # score above the group at 2.0 standard deviations, which therefore passes by four of theirs, and twice k keys do; at 1.8 26 +- 5.)
    ("long", wl.BF16, 9, 16, 2, 40000, 32, 300, 100, [(0.3, 2.0)]),
    ("long", wl.F16, 1, 1, 1, 100001, 256, 1000, 0, [(0.2, 2.0)]),
    ("long", wl.BF16, 1, 8, 1, 150000, 128, 1000, 30, [(0.2, 2.1)]),            # the row-tile scan
    ("long, tied", wl.BF16, 1, 8, 2, 131072, 256, 2048, 64, [(0.15, 3.0)]),
    ("long, tied", wl.F16, 16, 16, 4, 50000, 64, 500, 0, [(0.5, 2.8)]),         # one workgroup per head
    ("long, tied", wl.F16, 1, 8, 8, 100000, 64, 500, 0, [(0.7, 2.8)]),          # more ties than the boundary list holds: a fallback
    ("rescored", wl.F16, 1, 2, 1, 524288, 64, 1500, 0, [(0.92, 1.5)]),
    ("rescored", wl.BF16, 1, 1, 1, 524289, 256, 1500, 40, [(0.92, 1.5)]),
    ("rescored", wl.BF16, 1, 3, 1, 524000, 32, 1500, 0, [(0.92, 1.5)]),
    ("rescored", wl.F16, 3, 4, 1, 700000, 64, 1000, 50, [(0.8, 2.2)]),          # the row-tile scan, causal chunk
    ("row", wl.F16, 1, 2, 1, 524288, 128, 1500, 0, [(0.92, 3.0)]),             # more ties than the segments hold
])
def test_lists_that_do_not_fit(expect, dtype, M, Hq, Hkv, N, d, k, window, groups):
    q, K, V = (wl.quantize(a, dtype) for a in make_tied(N + k, M, Hq, Hkv, N, d, groups))
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, N, k, dtype, max_window=window, max_queries=M)
    try:
        cache.append(0, 0, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        qd = H.to_torch(q, dtype, DEV)[None].contiguous()
        res = cache.decode_multi(0, qd, k, window=window)
        fb = cache.last_fallbacks()
        how, want_fb = how_selected(cache, M * Hq)
        print(how[:8], "fallbacks", fb, flush=True)
        assert set(how) == {expect}
        assert fb == want_fb
        again = cache.decode_multi(0, qd, k, window=window)
        torch.cuda.synchronize()
        for a, b in zip(res, again):
            assert torch.equal(a, b)
        check_exact(tuple(t[0].cpu().numpy() for t in res), q, K, V, dtype, k, True, window, expect)
    finally:
        cache.close()


def test_a_segment_that_overflows_again():
    """512 of the best keys lie in the tiles of one wave segment, more than it holds, and still do when the bins
    below the k-th score's are left out: the head is selected from its full score row."""
    dtype, Hq, N, d, k, n_seg, sid = wl.F16, 2, 524288, 64, 1500, 1024, 517
    tiles = [i * n_seg + ((sid + (((i * 0x9E3779B1) & 0xFFFFFFFF) >> 12)) & (n_seg - 1)) for i in range(N // 64 // n_seg)]
    hot = np.concatenate([np.arange(t * 64, t * 64 + 64) for t in tiles])
    q, K, V = (wl.quantize(a, dtype) for a in make_tied(11, 1, Hq, 1, N, d, [], hot))
    cache = ta.TopkAttnCache(1, 1, Hq, 1, d, N, k, dtype)
    try:
        cache.append(0, 0, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        res = cache.decode_multi(0, H.to_torch(q, dtype, DEV)[None].contiguous(), k)
        assert cache.last_fallbacks() == Hq
        assert ta.topk_attn_debug_read_workspace_dims(cache.h)[4] == n_seg
        rec = ta.topk_attn_last_selection_records(cache.h, Hq)
        assert all(r[0] & 0xFF == 1 and r[0] >> 8 == 2 for r in rec), rec
        check_exact(tuple(t[0].cpu().numpy() for t in res), q, K, V, dtype, k, True, 0, "one hot segment")
    finally:
        cache.close()


@pytest.mark.parametrize("dtype,M,Hq,Hkv,N,d,k,window,index", [
    (wl.F16, 1, 2, 1, 300000, 128, 1500, 0, ta.INDEX_NONE),
    (wl.BF16, 1, 8, 2, 300000, 64, 800, 0, ta.INDEX_NONE),
    (wl.BF16, 1, 3, 1, 200000, 32, 500, 0, ta.INDEX_NONE),
    (wl.F16, 1, 4, 4, 150000, 256, 700, 100, ta.INDEX_NONE),
    (wl.F16, 1, 8, 1, 300000, 128, 1500, 0, ta.INDEX_NONE),        # the row-tile scan
    (wl.BF16, 1, 40, 2, 200000, 64, 600, 0, ta.INDEX_NONE),        # two row tiles
    (wl.F16, 4, 8, 2, 100001, 128, 700, 0, ta.INDEX_NONE),
    (wl.BF16, 16, 16, 4, 40000, 64, 400, 64, ta.INDEX_NONE),       # one workgroup per head
    (wl.BF16, 1, 4, 1, 30000, 128, 4000, 90, ta.INDEX_NONE),       # as many rows as fit
    (wl.F16, 1, 4, 1, 100000, 64, 700, 0, ta.INDEX_INT8),          # with an index: from the full score row
    (wl.BF16, 1, 4, 2, 70001, 256, 300, 64, ta.INDEX_INT8),
    (wl.F16, 1, 4, 2, 70000, 32, 500, 0, ta.INDEX_PAGES),
    (wl.BF16, 1, 6, 2, 50001, 128, 300, 200, ta.INDEX_PAGES),
])
def test_forced_redo_by_both_selections(dtype, M, Hq, Hkv, N, d, k, window, index):
    """Every head's list treated as unusable, by the one-launch selection (which these calls take) and by the chip-wide one: what the
    second scoring keeps is what the scan counted, and the selection is the oracle's."""
    q, K, V = (wl.quantize(a, dtype) for a in make_tied(N + k, M, Hq, Hkv, N, d, []))
    rows = M * Hq
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, N, k, dtype, max_window=window, max_queries=M, index_kind=index)
    try:
        cache.set_path({ta.INDEX_NONE: ta.PATH_AUTO, ta.INDEX_INT8: ta.PATH_INDEX, ta.INDEX_PAGES: ta.PATH_PAGES}[index])
        cache.append(0, 0, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        qd = H.to_torch(q, dtype, DEV)[None].contiguous()
        for mode in (1, 2):
            ta.topk_attn_debug_force_redo(cache.h, mode)
            res = cache.decode_multi(0, qd, k, window=window)
            assert cache.last_fallbacks() == 0          # forced, not counted
            rec = ta.topk_attn_last_selection_records(cache.h, rows)
            assert all(r[0] == (4 << 8 | (0 if index == ta.INDEX_NONE else 1)) for r in rec), rec
            handed_over = ta.topk_attn_debug_read_workspace(cache.h, "flags", np.uint32, rows) >> 8
            assert (handed_over > 0).all() if mode == 1 else (handed_over == 0).all()
            if index == ta.INDEX_NONE:
                dims = ta.topk_attn_debug_read_workspace_dims(cache.h)
                kept = ta.topk_attn_debug_read_workspace(cache.h, "seg_cnt2", np.uint32, dims[4] * rows).reshape(rows, dims[4])
                assert [int(c.sum()) for c in kept] == [r[1] + r[3] for r in rec]
            check_exact(tuple(t[0].cpu().numpy() for t in res), q, K, V, dtype, k, True, window, f"mode {mode}")
    finally:
        cache.close()


@pytest.mark.parametrize("dtype,d,window,one_launch", [(wl.BF16, 256, 1280, True), (wl.BF16, 256, 1281, False), (wl.F16, 128, 2561, False),
                                                       (wl.F16, 64, 3900, True)])
def test_wide_windows_go_to_the_chip_wide_selection(dtype, d, window, one_launch):
    """Every workgroup of the one-launch selection scores the whole window: both sides of the rule that bounds it."""
    Hq, Hkv, N, k = 8, 2, 40000, 150
    q, K, V = (wl.quantize(a, dtype) for a in make_tied(d + window, 1, Hq, Hkv, N, d, []))
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, N, k, dtype, max_window=window)
    try:
        cache.append(0, 0, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        res = cache.decode_multi(0, H.to_torch(q, dtype, DEV)[None].contiguous(), k, window=window)
        torch.cuda.synchronize()
        handed_over = ta.topk_attn_debug_read_workspace(cache.h, "flags", np.uint32, Hq) >> 8
        assert (handed_over > 0).all() if one_launch else (handed_over == 0).all()
        check_exact(tuple(t[0].cpu().numpy() for t in res), q, K, V, dtype, k, True, window, f"window {window}")
    finally:
        cache.close()


@pytest.mark.parametrize("N,filtered", [(16385, False), (24575, False), (24576, True)])
def test_pages_of_a_short_cache_are_not_filtered(N, filtered):
    """With a page index the filtered scan begins where it did without the one-launch selection."""
    dtype, Hq, Hkv, d, k = wl.F16, 8, 2, 128, 100
    q, K, V = (wl.quantize(a, dtype) for a in make_tied(N, 1, Hq, Hkv, N, d, []))
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, N, k, dtype, index_kind=ta.INDEX_PAGES)
    try:
        cache.set_path(ta.PATH_PAGES)
        cache.append(0, 0, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        res = cache.decode_multi(0, H.to_torch(q, dtype, DEV)[None].contiguous(), k)
        torch.cuda.synchronize()
        assert (ta.topk_attn_debug_read_workspace_dims(cache.h)[4] > 0) == filtered
        check_exact(tuple(t[0].cpu().numpy() for t in res), q, K, V, dtype, k, True, 0, f"N={N}")
    finally:
        cache.close()


@pytest.mark.parametrize("B,M,Hq,Hkv,N,d,k,window", [
    (9, 1, 32, 8, 26000, 64, 500, 0),                # more heads than compute units, the second round nearly empty
    (17, 1, 32, 4, 25601, 128, 300, 0),              # row tiles, more than two workgroups a compute unit
    (9, 1, 32, 8, 27000, 64, 300, 100),
    (1, 14, 32, 8, 30001, 128, 500, 0),
    (1, 25, 32, 8, 26000, 64, 700, 64),
    (3, 3, 36, 9, 26000, 32, 200, 0),
])
def test_more_heads_than_compute_units_one_launch(B, M, Hq, Hkv, N, d, k, window):
    """Lists of any number of heads beyond the compute units, ragged sequences: the records say that all of k is certain."""
    dtype = wl.F16
    n = [N] + [N - 3001 * (b % 4) - 7 * b for b in range(1, B)]
    if B > 2:
        n[1] = k + window + 50                       # a sequence too short to filter rides along
    data = [tuple(wl.quantize(a, dtype) for a in make_tied(N + b, M, Hq, Hkv, n[b], d, [])) for b in range(B)]
    cache = ta.TopkAttnCache(1, B, Hq, Hkv, d, N, k, dtype, max_queries=M, max_window=window)
    try:
        for b, (q, K, V) in enumerate(data):
            cache.append(0, b, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        qd = torch.stack([H.to_torch(x[0], dtype, DEV) for x in data]).contiguous()
        res = cache.decode_multi(0, qd, k, causal=True, window=window)
        torch.cuda.synchronize()
        rec = ta.topk_attn_last_selection_records(cache.h, B * M * Hq)
        assert all(r[1] == k and r[2] == 0 for r in rec[:M * Hq])
        for b in sorted({0, 1 % B, B - 1}):
            q, K, V = data[b]
            check_exact(tuple(t[b].cpu().numpy() for t in res), q, K, V, dtype, k, True, window, f"seq {b}")
    finally:
        cache.close()


@pytest.mark.parametrize("B,M,Hq,Hkv,N,d,k", [
    (1, 15, 32, 8, 25000, 128, 500),
    (1, 14, 32, 8, 25000, 128, 500),
    (1, 12, 32, 8, 25000, 64, 500),
    (1, 25, 32, 8, 25000, 64, 500),
    (9, 1, 32, 8, 16000, 64, 500),                   # a batch
    (9, 1, 32, 8, 16600, 256, 4096),                 # as many rows as one launch takes
    (1, 9, 32, 8, 16385, 128, 300),                  # the shortest chunk that is filtered
])
def test_more_heads_than_compute_units(B, M, Hq, Hkv, N, d, k):
    """The one-launch selection takes the lists of calls of more than 256 heads whatever their length: the records say that all of k is certain."""
    dtype = wl.BF16
    data = [tuple(wl.quantize(a, dtype) for a in make_tied(N + b, M, Hq, Hkv, N, d, [])) for b in range(B)]
    cache = ta.TopkAttnCache(1, B, Hq, Hkv, d, N, k, dtype, max_queries=M)
    try:
        for b, (q, K, V) in enumerate(data):
            cache.append(0, b, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        qd = torch.stack([H.to_torch(x[0], dtype, DEV) for x in data]).contiguous()
        res = cache.decode_multi(0, qd, k)
        torch.cuda.synchronize()
        rec = ta.topk_attn_last_selection_records(cache.h, B * M * Hq)
        assert all(r[1] == k and r[2] == 0 for r in rec)
        for b in sorted({0, B - 1}):
            q, K, V = data[b]
            check_exact(tuple(t[b].cpu().numpy() for t in res), q, K, V, dtype, k, True, 0, f"seq {b}")
    finally:
        cache.close()


@pytest.mark.parametrize("dtype,M,Hq,Hkv,N,d,k,window,run,spread", [
    (wl.F16, 1, 8, 2, 60000, 128, 900, 0, 1, 3),           # hundreds of distinct scores in the k-th score's bin, 1024 threads
    (wl.BF16, 17, 16, 4, 50000, 64, 500, 40, 1, 3),        # 512 threads
    (wl.F16, 1, 4, 1, 100000, 64, 700, 0, 1, 1),           # 1024 segments
    (wl.F16, 1, 4, 1, 100000, 64, 700, 0, 64, 3),          # whole tiles of candidates: deep segments, few entries
    (wl.BF16, 17, 16, 4, 50000, 32, 150, 0, 64, 3),
    (wl.F16, 1, 8, 8, 80000, 256, 400, 100, 64, 2),
    (wl.F16, 1, 8, 2, 60000, 128, 900, 0, 1, 0),           # all of them equal
    (wl.BF16, 17, 16, 4, 50000, 64, 500, 0, 64, 0),
])
def test_crowded_bins_and_sparse_lists(dtype, M, Hq, Hkv, N, d, k, window, run, spread):
    """1.4 k keys in runs of `run` score alike but for steps in `spread` channels, around the k-th score."""
    q, K, V = make_tied(N + k + run, M, Hq, Hkv, N, d, [])
    g = np.random.default_rng(k)
    sigma = np.sqrt((17.0 ** 2 - 1) / 12)
    for h in range(Hkv):
        Q = q[0, h * (Hq // Hkv):(h + 1) * (Hq // Hkv)].astype(np.float64)
        at = np.rint(8 * np.linalg.lstsq(Q, 3.0 * sigma * np.linalg.norm(Q, axis=1), rcond=None)[0]) / 8
        starts = g.permutation((N - window) // run - 1)[:-(-7 * k // (5 * run))] * run
        hot = (starts[:, None] + np.arange(run)).ravel()
        K[h, hot] = at
        for c in g.permutation(d)[:spread]:
            K[h, hot, c] += g.integers(-8, 9, hot.size) / 8
    q, K, V = (wl.quantize(a, dtype) for a in (q, K, V))
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, N, k, dtype, max_window=window, max_queries=M)
    try:
        cache.append(0, 0, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        qd = H.to_torch(q, dtype, DEV)[None].contiguous()
        res = cache.decode_multi(0, qd, k, window=window)
        assert cache.last_fallbacks() == 0
        rows = M * Hq
        in_bin = max(r[3] for r in ta.topk_attn_last_selection_records(cache.h, rows))
        n_seg = ta.topk_attn_debug_read_workspace_dims(cache.h)[4]
        cnt = ta.topk_attn_debug_read_workspace(cache.h, "seg_cnt", np.uint32, n_seg * rows).reshape(rows, n_seg)
        threads = 512 if rows > 256 else 1024
        deep = (-(-cnt.max(1).astype(int) // 16) * 16 * n_seg > 8 * threads) & (cnt.sum(1) + in_bin <= min(8 * threads, 3584 if threads == 512 else 10240))
        print("in the bin", in_bin, "segments", n_seg, "deep lists", deep.sum(), "of", rows, flush=True)
        assert in_bin > 256 or run > 1
        assert deep.any() or run == 1
        again = cache.decode_multi(0, qd, k, window=window)
        torch.cuda.synchronize()
        for a, b in zip(res, again):
            assert torch.equal(a, b)
        check_exact(tuple(t[0].cpu().numpy() for t in res), q, K, V, dtype, k, True, window, "crowded")
    finally:
        cache.close()


@pytest.mark.parametrize("M,Hq,Hkv,N,d,k,bound", [(16, 32, 8, 40000, 128, 2048, 1.5e-7), (20, 16, 4, 30000, 256, 2000, 1.7e-7)])
def test_sums_of_workgroups_with_512_threads(M, Hq, Hkv, N, d, k, bound):
    """Relative error (2-norm) of the weighted sum of the selected value rows against 64 bits, for more heads than compute units.  Bounds:
    half way between the sums a lane makes of every fourth row (1.3e-7 and 1.4e-7 measured) and one sum of all its rows (1.75e-7 and
    2.2e-7), whose rounding errors grow with the length of the chain (64 and 125 rows)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, N, k, wl.F16, max_queries=M)
    try:
        K, V = (torch.randn((Hkv, N, d), generator=g, device=DEV).half() for _ in range(2))
        cache.append(0, 0, K, V, head_major=True)
        q = (torch.randn((1, M, Hq, d), generator=g, device=DEV) * 0.3).half()
        out, idx, vals, _ = cache.decode_multi(0, q, k)
        torch.cuda.synchronize()
        w = torch.softmax(vals[0].double() / d ** 0.5, -1)
        ref = torch.stack([(w[:, h, :, None] * V[h * Hkv // Hq].double()[idx[0, :, h].long()]).sum(1) for h in range(Hq)], 1)
        err = ((out[0].double() - ref).norm() / ref.norm()).item()
        print("error", err, flush=True)
        assert err < bound
    finally:
        cache.close()


def test_many_tied_candidates_fit_the_list():
    """16 sequences of 60000 tokens, k = 1000, 8 KV heads: a list holds 39000 keys that tie above the threshold (3072 entries in each
    of its 16 segments)."""
    B, Hq, Hkv, N, d, k = 16, 8, 8, 60000, 32, 1000
    q, K, V = (wl.quantize(a, wl.F16) for a in make_tied(5, 1, Hq, Hkv, N, d, [(0.65, 1.5)]))
    cache = ta.TopkAttnCache(1, B, Hq, Hkv, d, N, k, wl.F16)
    try:
        Kd, Vd = H.to_torch(K, wl.F16, DEV), H.to_torch(V, wl.F16, DEV)
        for b in range(B):
            cache.append(0, b, Kd if b == 3 else torch.randn_like(Kd), Vd, head_major=True)
        qd = H.to_torch(q, wl.F16, DEV)[None].repeat(B, 1, 1, 1).contiguous()
        res = cache.decode_multi(0, qd, k)
        assert cache.last_fallbacks() == 0
        dims = ta.topk_attn_debug_read_workspace_dims(cache.h)
        cnt = ta.topk_attn_debug_read_workspace(cache.h, "seg_cnt", np.uint32, dims[4] * B * Hq).reshape(B, Hq, dims[4])
        assert (cnt[3].sum(1) >= 39000).all() and cnt[3].max() <= dims[5]
        rec = ta.topk_attn_last_selection_records(cache.h, B * Hq)       # (lists of any length are reported alike)
        assert all(r[0] == 0 and r[1] == k and r[2] == 0 for r in rec)
        check_exact(tuple(t[3].cpu().numpy() for t in res), q, K, V, wl.F16, k, True, 0, "tied")
    finally:
        cache.close()


@pytest.mark.parametrize("N,n_seg", [(131072, 128), (98304, 128), (98000, 64)])
def test_split_of_three_row_blocks(N, n_seg):
    """17 queries, 8 KV heads: 24 streams of row blocks, split until their workgroups fill the chip while a wave keeps a dozen tiles."""
    dtype, M, Hq, Hkv, d, k = wl.F16, 17, 32, 8, 32, 400
    q, K, V = (wl.quantize(a, dtype) for a in make_tied(N, M, Hq, Hkv, N, d, []))
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, N, k, dtype, max_queries=M)
    try:
        cache.append(0, 0, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
        res = cache.decode_multi(0, H.to_torch(q, dtype, DEV)[None].contiguous(), k)
        torch.cuda.synchronize()
        assert ta.topk_attn_debug_read_workspace_dims(cache.h)[4] == n_seg
        assert cache.last_fallbacks() == 0
        check_exact(tuple(t[0].cpu().numpy() for t in res), q, K, V, dtype, k, True, 0, f"N={N}")
    finally:
        cache.close()
