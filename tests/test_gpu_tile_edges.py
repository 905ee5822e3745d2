"""The tile that the end of a cache cuts short, in every scan over 16-bit keys and over codes: the last rows are not missed and
the slots behind the end are no keys.  Those slots hold NaN ("mixed"), which would show in a result, or zeros under keys whose scores are
all negative ("negative"), so that a slot taken for a key, read from memory or as the zeros of a bounded load, would be selected.  Elements
of q and K are small integers, so scores are exact in fp32 and the selection has to equal the oracle's."""
import numpy as np
import pytest
import torch

import helpers as H
from oracle import c_oracle
from paper_2502_06766_amd import topk_attn as ta
from paper_2502_06766_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0) if torch.cuda.is_available() else None
PATHS = {"filter": ta.PATH_FILTER, "full": ta.PATH_FULL, "auto": ta.PATH_AUTO}


@pytest.mark.parametrize("scores", ["mixed", "negative"])
@pytest.mark.parametrize("d", [32, 64, 128, 256])
@pytest.mark.parametrize("path,Hq,Hkv,seqs", [
    ("filter", 4, 1, 1), ("filter", 6, 2, 3), ("filter", 8, 1, 1), ("filter", 20, 1, 2), ("full", 4, 1, 1), ("full", 16, 2, 2), ("auto", 4, 2, 3),
])
def test_rows_behind_the_end_of_the_cache(d, path, Hq, Hkv, seqs, scores):
    g = np.random.default_rng(d + Hq)
    for n0 in (300, 1983, 5000):                                      # (auto: the one launch over short sequences up to 512)
        lens = [n0 // 64 * 64 + r for r in (1, 63, 16, 17, 0)]
        if path == "auto":
            lens = [n % 448 + 20 for n in lens]
        for n in (lens if seqs == 1 else [lens]):
            ns = [n] if seqs == 1 else n[:seqs]
            k = 20
            cache = ta.TopkAttnCache(1, seqs, Hq, Hkv, d, max(ns) + 130, k, wl.F16)
            try:
                neg = scores == "negative"
                cache.kv.fill_(0 if neg else 0xFF)                    # (0xFFFF: NaN)
                data = []
                q = wl.quantize(g.integers(1 if neg else -3, 4, (seqs, Hq, d)).astype(np.float32), wl.F16)
                for b, nb in enumerate(ns):
                    K = wl.quantize(g.integers(-8, 0 if neg else 9, (Hkv, nb, d)).astype(np.float32), wl.F16)
                    if neg:
                        K[:, -1, 1:] = 0                              # the last key is the best there is, and below zero
                    else:
                        K[:, -1] = 8 * np.sign(q[b].reshape(Hkv, -1, d)[:, 0])       # the last key is a winner of the group's first head
                    V = wl.quantize(g.standard_normal((Hkv, nb, d)).astype(np.float32), wl.F16)
                    cache.append(0, b, H.to_torch(K, wl.F16, DEV), H.to_torch(V, wl.F16, DEV), head_major=True)
                    data.append((K, V))
                cache.set_path(PATHS[path])
                res = cache.decode(0, H.to_torch(q, wl.F16, DEV), k)
                torch.cuda.synchronize()
                for b, (K, V) in enumerate(data):
                    assert int(res[1][b].max()) < ns[b] and (not neg or (res[1][b] == ns[b] - 1).any(1).all())
                    ref = c_oracle.topk_attention(q[b], K, V, wl.F16, k)
                    H.check_against_oracle(*(r[b].cpu().numpy() for r in res), ref, np.full(Hq, 1e-30), min(k, ns[b]), H.out_tolerance(wl.F16),
                                           float(np.abs(wl.widen(V, wl.F16)).max()), f"d={d} {path} n={ns[b]}")
            finally:
                cache.close()


@pytest.mark.parametrize("scores", ["mixed", "negative"])
@pytest.mark.parametrize("d,n", [(64, 20001), (128, 17023), (128, 16448), (256, 17040)])
def test_codes_behind_the_end_of_the_cache(d, n, scores):
    """The same through the int8 index (codes of -1 and scales of NaN behind the end, or zeros under negative scores): the k keys far above
    all others, the last one among them, are found."""
    neg = scores == "negative"
    g = np.random.default_rng(d + n)
    Hkv, k = 3, 20
    q = g.integers(1, 4, (Hkv, d)).astype(np.float32) * g.choice([-1.0, 1.0], (Hkv, d)).astype(np.float32)
    Kf = g.integers(2, 5, (Hkv, n, d)) * -np.sign(q)[:, None] if neg else g.integers(-2, 3, (Hkv, n, d))
    Kf = Kf.astype(np.float32)
    for h in range(Hkv):
        pos = np.append(g.permutation(n - 1)[:k - 1], n - 1)
        for i, p in enumerate(pos):                                   # (scores that differ)
            Kf[h, p] = -np.sign(q[h]) if neg else 8 * np.sign(q[h])
            Kf[h, p, slice(i + 1, None) if neg else slice(i)] = 0
    q, K = wl.quantize(q, wl.F16), wl.quantize(Kf, wl.F16)
    V = wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), wl.F16)
    cache = ta.TopkAttnCache(1, 1, Hkv, Hkv, d, n + 130, k, wl.F16, index_kind=ta.INDEX_INT8)
    try:
        cache.kv.fill_(0 if neg else 0xFF)
        cache.append(0, 0, H.to_torch(K, wl.F16, DEV), H.to_torch(V, wl.F16, DEV), head_major=True)
        cache.set_path(ta.PATH_INDEX)
        res = cache.decode(0, H.to_torch(q[None], wl.F16, DEV), k)
        torch.cuda.synchronize()
        assert int(res[1].max()) < n
        H.check_against_oracle(*(r[0].cpu().numpy() for r in res), c_oracle.topk_attention(q, K, V, wl.F16, k), np.full(Hkv, 1e-30), k,
                               H.out_tolerance(wl.F16), float(np.abs(wl.widen(V, wl.F16)).max()), f"int8 d={d} n={n}")
        assert cache.last_fallbacks() == 0
    finally:
        cache.close()


@pytest.mark.parametrize("d,Hq,Hkv,n", [(64, 4, 1, 40001), (128, 8, 2, 34023), (256, 3, 1, 37072), (32, 4, 2, 33000)])
def test_pages_behind_the_end_of_the_cache(d, Hq, Hkv, n):
    """The same through the page index: negative scores, a cut-short last page, and pages that are ruled out (the search took that path)."""
    g = np.random.default_rng(d + n)
    k = 20
    q = wl.quantize(g.integers(1, 4, (Hq, d)).astype(np.float32), wl.F16)
    Kf = g.integers(-2, 0, (Hkv, n, d)).astype(np.float32)
    Kf[:, :n // 2] -= 100                                             # half the pages lie far below
    Kf[:, -1, 1:] = 0
    K, V = wl.quantize(Kf, wl.F16), wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), wl.F16)
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, n + 130, k, wl.F16, index_kind=ta.INDEX_PAGES)
    try:
        cache.kv.zero_()
        cache.append(0, 0, H.to_torch(K, wl.F16, DEV), H.to_torch(V, wl.F16, DEV), head_major=True)
        cache.set_path(ta.PATH_PAGES)
        res = cache.decode(0, H.to_torch(q[None], wl.F16, DEV), k)
        torch.cuda.synchronize()
        read, total = ta.topk_attn_last_pages_read(cache.h)
        assert 0 < read < total
        assert int(res[1].max()) < n and (res[1][0] == n - 1).any(1).all()
        H.check_against_oracle(*(r[0].cpu().numpy() for r in res), c_oracle.topk_attention(q, K, V, wl.F16, k), np.full(Hq, 1e-30), k,
                               H.out_tolerance(wl.F16), float(np.abs(wl.widen(V, wl.F16)).max()), f"pages d={d} n={n}")
    finally:
        cache.close()


@pytest.mark.parametrize("d,Hq,Hkv,n,k", [(64, 4, 1, 20001, 16), (64, 2, 2, 33000, 9000), (128, 4, 1, 17023, 1500), (128, 8, 8, 30000, 4000),
                                          (256, 3, 1, 18000, 3000), (256, 8, 4, 25001, 300)])
def test_exact_scores_of_coded_candidates(d, Hq, Hkv, n, k):
    """Segments of a few candidates and of several hundred (rounds of 8 to 32 rows, batches of 64): every score that leaves the
    index path is the exact product of its row, which integers make the same in any order of the sum."""
    g = np.random.default_rng(d + n)
    qi = g.integers(-3, 4, (Hq, d)).astype(np.float32)
    Ki = g.integers(-8, 9, (Hkv, n, d)).astype(np.float32)
    q, K = wl.quantize(qi, wl.BF16), wl.quantize(Ki, wl.BF16)
    V = wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), wl.BF16)
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, n, k, wl.BF16, index_kind=ta.INDEX_INT8)
    try:
        cache.append(0, 0, H.to_torch(K, wl.BF16, DEV), H.to_torch(V, wl.BF16, DEV), head_major=True)
        cache.set_path(ta.PATH_INDEX)
        _, idx, vals, _ = cache.decode(0, H.to_torch(q[None], wl.BF16, DEV), k)
        idx, vals = idx[0].cpu().numpy(), vals[0].cpu().numpy()
        for h in range(Hq):
            s = Ki[h // (Hq // Hkv)] @ qi[h]                          # (integers below 2^24: exact)
            assert len(set(idx[h].tolist())) == k
            assert np.array_equal(vals[h], s[idx[h]])
            assert np.mean(vals[h] >= np.sort(s)[-k]) > 0.98          # coding noise: 0.4 % of a row's largest element per channel
    finally:
        cache.close()


@pytest.mark.parametrize("M,Hq,Hkv", [(1, 5, 1), (1, 16, 1), (1, 17, 1), (4, 8, 1), (11, 3, 1), (3, 16, 2)])
@pytest.mark.parametrize("d,n,k,window,keys", [(64, 1991, 40, 0, "equal"), (64, 3000, 700, 9, "runs"), (128, 2049, 5, 0, "runs"), (128, 1983, 1500, 0, "random"),
                                               (256, 1100, 64, 70, "runs"), (64, 2400, 49, 0, "runs"), (64, 2400, 50, 0, "runs"), (32, 2401, 50, 5, "equal"), (32, 2400, 600, 5, "equal")])
def test_row_tiles_filter(d, n, k, window, keys, M, Hq, Hkv):
    """What passes the row-tile filter: everything (tied keys, every lane's mask full and the stages flushed at each tile), runs of
    64 and more high scores, few; k on both sides of where what passes is staged another way (48 k = n); with prefixes of a causal chunk that
    end within a tile.  Integers, so the selected scores are exact."""
    g = np.random.default_rng(d + n + Hq)
    qi = g.integers(1, 4, (M, Hq, d)).astype(np.float32)
    Ki = g.integers(-8, 9, (Hkv, n, d)).astype(np.float32)
    if keys == "equal":
        Ki[:] = Ki[:, :1]
    elif keys == "runs":
        for lo in range(100, n - 150, 701):
            Ki[:, lo:lo + 130] = np.abs(Ki[:, lo:lo + 130])           # (q is positive)
    q, K = wl.quantize(qi, wl.BF16), wl.quantize(Ki, wl.BF16)
    V = wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), wl.BF16)
    cache = ta.TopkAttnCache(1, 1, Hq, Hkv, d, n, k, wl.BF16, max_window=window, max_queries=M)
    try:
        cache.append(0, 0, H.to_torch(K, wl.BF16, DEV), H.to_torch(V, wl.BF16, DEV), head_major=True)
        cache.set_path(ta.PATH_FILTER)
        qd = H.to_torch(q, wl.BF16, DEV)[None].contiguous()
        if M > 1:
            out, idx, vals, _ = cache.decode_multi(0, qd, k, causal=True, window=window)
        else:
            out, idx, vals, _ = (r[:, None] for r in cache.decode(0, qd[:, 0].contiguous(), k, window=window))
        out, idx, vals = (r[0].cpu().numpy() for r in (out, idx, vals))
        Vf = wl.widen(V, wl.BF16).astype(np.float64)
        for m in range(M):
            p = n - (M - 1 - m)
            for h in range(Hq):
                s = Ki[h // (Hq // Hkv), :p].astype(np.float64) @ qi[m, h]
                sel = idx[m, h]
                assert len(set(sel.tolist())) == k and sel.min() >= 0 and sel.max() < p - window
                assert np.array_equal(vals[m, h], s[sel])
                assert np.array_equal(np.sort(vals[m, h]), np.sort(s[:p - window])[-k:])
                pos = np.concatenate([sel, np.arange(p - window, p)])
                w = np.exp((s[pos] - s[pos].max()) / np.sqrt(d))
                ref = (w[:, None] * Vf[h // (Hq // Hkv), pos]).sum(0) / w.sum()
                # sums of up to 1570 terms in 32 bits, weights by a base-2 exponential
                assert np.abs(out[m, h] - ref).max() < 1e-5 * np.abs(Vf).max()
    finally:
        cache.close()
