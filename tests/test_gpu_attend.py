"""Selection and attention of a head in one launch (csrc/attend.hip), over score rows and over candidate lists, at the
sizes where a branch of its dispatch begins or ends, against the oracle.  The bars are those of the other
parity tests: sets equal to the oracle's up to keys within fp32 rounding of the k-th score (exactly
equal where the scores are exact in fp32), outputs within the usual tolerance, repeated calls bit-identical."""
import numpy as np
import pytest
import torch

import helpers as H
from oracle import c_oracle
from paper_2502_06766_amd import topk_attn as ta
from paper_2502_06766_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0) if torch.cuda.is_available() else None


def _make(dtype, B, Hq, Hkv, N, d, seed):
    g = np.random.default_rng(seed)
    lens = [max(1, N - (37 * b) % max(1, N // 2)) for b in range(B)]
    q = wl.quantize(g.standard_normal((B, Hq, d)).astype(np.float32), dtype)
    K = [wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), dtype) for n in lens]
    V = [wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), dtype) for n in lens]
    return q, K, V


def _decode(q, K, V, dtype, k, window=0, path=ta.PATH_AUTO, N=None, calls=2):
    """Decodes a batch twice (the results must be bit-identical) and returns numpy (out, idx, vals, lse)."""
    B, Hq, d = q.shape
    cache = ta.TopkAttnCache(1, B, Hq, K[0].shape[0], d, N or max(x.shape[1] for x in K), k, dtype, max_window=window)
    try:
        cache.set_path(path)
        for b in range(B):
            cache.append(0, b, H.to_torch(K[b], dtype, DEV), H.to_torch(V[b], dtype, DEV), head_major=True)
        qd = H.to_torch(q, dtype, DEV)
        res = [cache.decode(0, qd, k, window=window) for _ in range(calls)]
        torch.cuda.synchronize()
        for r in res[1:]:
            for a, b in zip(res[0], r):
                assert torch.equal(a, b)
        return tuple(t.cpu().numpy() for t in res[0])
    finally:
        cache.close()


@pytest.mark.parametrize("dtype,B,Hq,Hkv,N,d,k,window", [
    (wl.F32, 1, 1, 1, 1, 64, 1, 0),
    (wl.F32, 1, 1, 1, 1025, 128, 1024, 0),
    (wl.F16, 1, 8, 2, 63, 32, 100, 0),               # k beyond the cache
    (wl.BF16, 1, 4, 2, 4096, 128, 4096, 0),          # everything selected, as many rows as fit
    (wl.F16, 1, 4, 1, 4097, 256, 77, 4019),          # rows of the selection and the window fill the list
    (wl.F16, 1, 4, 1, 4097, 64, 78, 4019),           # one row too many: the general path's other back end
    (wl.BF16, 1, 6, 2, 8193, 64, 1, 0),
    (wl.F32, 1, 4, 2, 16384, 64, 300, 100),
    (wl.F16, 1, 32, 8, 16384, 128, 4000, 0),
    (wl.F16, 1, 12, 2, 16385, 128, 500, 33),         # one score too many for a row: filtered scan and candidate list
    (wl.F32, 1, 4, 2, 16385, 128, 500, 0),           # the same in fp32: no filtered scan
    (wl.BF16, 40, 8, 2, 2048, 64, 200, 16),          # more heads than compute units: small workgroups
    (wl.F16, 40, 8, 2, 2049, 128, 600, 0),
    (wl.F32, 70, 4, 2, 4096, 64, 1024, 0),
    (wl.BF16, 36, 8, 4, 4097, 64, 64, 5),
    (wl.F16, 33, 8, 4, 8192, 32, 2048, 0),
    (wl.F16, 3, 64, 8, 30001, 64, 900, 0),           # candidate lists, 192 heads: one workgroup each
    (wl.BF16, 2, 8, 2, 40000, 128, 1500, 700),       # candidate lists, eight workgroups per head, window
    (wl.F16, 1, 2, 1, 50000, 256, 4096, 0),          # as many rows as fit beside a list
])
def test_sizes_at_the_edges(dtype, B, Hq, Hkv, N, d, k, window):
    q, K, V = _make(dtype, B, Hq, Hkv, N, d, seed=N + k)
    res = _decode(q, K, V, dtype, k, window)
    for b in sorted({0, B // 2, B - 1}):
        H.check_unmargined(tuple(r[b] for r in res), q[b], K[b], V[b], dtype, k, window, f"N={N} k={k} seq {b}")


@pytest.mark.parametrize("dtype,B,Hq,Hkv,N,d,k", [
    (wl.F16, 2, 4, 1, 1, 64, 1),                     # one token
    (wl.BF16, 1, 3, 3, 65, 32, 90),                  # k beyond the cache, a second tile of one key
    (wl.F16, 3, 8, 2, 512, 128, 512),                # everything selected, as many rows as fit
    (wl.F16, 3, 8, 2, 512, 128, 513),                # one too many: rows and scores in two launches
    (wl.BF16, 32, 16, 4, 1024, 128, 100),            # 128 streams
    (wl.F16, 32, 24, 8, 1025, 64, 512),              # 256 streams, groups of three
    (wl.BF16, 32, 8, 8, 2048, 256, 33),              # groups of one
    (wl.F16, 64, 8, 4, 2049, 32, 256),
    (wl.BF16, 64, 16, 4, 4096, 64, 256),
    (wl.BF16, 64, 8, 4, 4097, 64, 256),              # one token too many
])
def test_short_sequences_in_one_launch(dtype, B, Hq, Hkv, N, d, k):
    q, K, V = _make(dtype, B, Hq, Hkv, N, d, seed=N + k + B)
    res = _decode(q, K, V, dtype, k)
    for b in sorted({0, B // 2, B - 1}):
        H.check_unmargined(tuple(r[b] for r in res), q[b], K[b], V[b], dtype, k, 0, f"N={N} k={k} seq {b}")


def test_short_sequences_with_ties():
    """Hundreds of equal scores per head, more than a wave ranks at once: the bins go on over the positions."""
    g = np.random.default_rng(17)
    dtype, B, Hq, Hkv, N, d, k = wl.F16, 64, 16, 4, 3000, 64, 200
    q = wl.quantize(g.integers(-1, 2, (B, Hq, d)).astype(np.float32), dtype)
    q[1] = 0                                         # all scores of a sequence equal
    K = [wl.quantize(g.integers(-1, 2, (Hkv, N, d)).astype(np.float32), dtype) for _ in range(B)]
    V = [wl.quantize(g.standard_normal((Hkv, N, d)).astype(np.float32), dtype) for _ in range(B)]
    res = _decode(q, K, V, dtype, k)
    for b in (0, 1, 63):
        ref = c_oracle.topk_attention(q[b], K[b], V[b], dtype, k)
        H.check_against_oracle(*(r[b] for r in res), ref, np.full(Hq, 1e-30), k, H.out_tolerance(dtype),
                               float(np.abs(wl.widen(V[b], dtype)).max()), f"seq {b}")


@pytest.mark.parametrize("path,dtype,N,k", [(ta.PATH_FULL, wl.F16, 9000, 2500), (ta.PATH_FULL, wl.F32, 3000, 5),
                                            (ta.PATH_FILTER, wl.F16, 9000, 1300), (ta.PATH_FILTER, wl.BF16, 120000, 300)])
@pytest.mark.parametrize("spread", [0, 1])
def test_ties_go_to_the_lower_position(path, dtype, N, k, spread):
    """All scores equal, or integer scores with hundreds of ties: the bins go on over the positions.  (120000 equal
    scores: the list is unusable, the head's workgroups score its keys again.)"""
    g = np.random.default_rng(N + k + spread)
    Hq, Hkv, d = 4, 2, 64
    q = wl.quantize(g.integers(-spread, spread + 1, (1, Hq, d)).astype(np.float32), dtype)
    K = [wl.quantize(g.integers(-spread, spread + 1, (Hkv, N, d)).astype(np.float32), dtype)]
    V = [wl.quantize(g.standard_normal((Hkv, N, d)).astype(np.float32), dtype)]
    out, idx, vals, lse = _decode(q, K, V, dtype, k, path=path)
    ref = c_oracle.topk_attention(q[0], K[0], V[0], dtype, k)
    H.check_against_oracle(out[0], idx[0], vals[0], lse[0], ref, np.full(Hq, 1e-30), k, H.out_tolerance(dtype),
                           float(np.abs(wl.widen(V[0], dtype)).max()), "ties")


@pytest.mark.parametrize("log2", [60, -70])
@pytest.mark.parametrize("N", [3000, 12000])
def test_scores_beyond_fp32_arithmetic(log2, N):
    """Scores whose range overflows fp32 (integers times 2^120 of either sign), or lies among the denormals (times
    2^-140): the bins are laid over the order-preserving keys instead.  The scores are exact, so is the selection."""
    g = np.random.default_rng(N)
    d, k = 64, 700
    q, K = np.zeros((1, 1, d), np.float32), np.zeros((1, N, d), np.float32)
    q[0, 0, 0] = 2.0 ** log2
    K[0, :, 0] = g.integers(-200, 201, N).astype(np.float32) * np.float32(2.0 ** log2)
    V = g.standard_normal((1, N, d)).astype(np.float32)
    out, idx, vals, _ = _decode(q, [K], [V], wl.F32, k)
    r_out, r_idx, r_vals, _ = c_oracle.topk_attention(q[0], K, V, wl.F32, k)
    assert np.array_equal(np.sort(idx[0, 0]), np.sort(r_idx[0]))
    assert np.array_equal(np.sort(vals[0, 0]), np.sort(r_vals[0]).astype(np.float32))
    np.testing.assert_allclose(out[0], r_out, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("dtype,N,k,window", [(wl.F16, 10000, 200, 30), (wl.BF16, 60000, 500, 64)])
def test_replays_of_a_captured_call_equal_eager_calls(dtype, N, k, window):
    """Rows and lists under graph capture: the shares of a head are counted in a word that every call clears again."""
    q, K, V = _make(dtype, 1, 8, 2, N, 64, seed=N)
    cache = ta.TopkAttnCache(1, 1, 8, 2, 64, N, k, dtype, max_window=window)
    try:
        cache.append(0, 0, H.to_torch(K[0], dtype, DEV), H.to_torch(V[0], dtype, DEV), head_major=True)
        qd = H.to_torch(q, dtype, DEV)
        out = torch.empty((1, 8, 64), dtype=torch.float32, device=DEV)
        idx = torch.empty((1, 8, k), dtype=torch.int32, device=DEV)
        s = torch.cuda.Stream()
        call = lambda: ta.topk_attn_decode_window(cache.h, 0, qd.data_ptr(), k, window, out.data_ptr(), idx.data_ptr(),
                                                  stream=s.cuda_stream)
        with torch.cuda.stream(s):
            call()
            s.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                call()
            for rep in range(4):
                qd.copy_(torch.roll(qd, 1, dims=1))
                out.zero_(); idx.zero_()
                g.replay()
                s.synchronize()
                got = out.clone(), idx.clone()
                eager = cache.decode(0, qd, k, window=window)
                s.synchronize()
                assert torch.equal(got[0], eager[0]) and torch.equal(got[1], eager[1]), f"replay {rep}"
    finally:
        cache.close()


@pytest.mark.parametrize("dtype,B,N,k,far", [(wl.F16, 1, 16384, 256, 3000.0), (wl.BF16, 1, 8000, 1000, 1000.0), (wl.F32, 1, 5000, 300, 30000.0),
                                              (wl.F16, 64, 4000, 100, 3000.0), (wl.BF16, 40, 3000, 600, -3000.0)])
def test_a_key_far_from_the_rest(dtype, B, N, k, far):
    """One key scores hundreds of standard deviations away from all others (an attention sink): the linear bins over the range leave
    most scores in one bin, which is split again."""
    q, K, V = _make(dtype, B, 8, 2, N, 64, seed=N + k)
    for b in range(B):
        Kf = wl.widen(K[b], dtype).astype(np.float32).copy()
        qf = wl.widen(q[b], dtype).astype(np.float32).reshape(2, 4, 64)
        Kf[:, 5] = far / 64 * qf.mean(axis=1)
        K[b] = wl.quantize(Kf, dtype)
    res = _decode(q, K, V, dtype, k)
    for b in sorted({0, B // 2, B - 1}):
        H.check_unmargined(tuple(r[b] for r in res), q[b], K[b], V[b], dtype, k, 0, f"far {far} seq {b}")


@pytest.mark.parametrize("dtype,B,Hq,Hkv,N,d,k,window", [
    (wl.F16, 1, 4, 2, 4096, 256, 3072, 0),           # 1.5 MB of value rows per head: one launch
    (wl.F16, 1, 4, 2, 4096, 256, 3073, 0),           # radix select and gather
    (wl.F32, 1, 4, 2, 5000, 256, 2048, 0),
    (wl.F32, 1, 4, 2, 5000, 256, 1849, 200),
    (wl.BF16, 5, 32, 8, 4000, 128, 1000, 0),         # 160 heads: a quarter of the row
    (wl.F16, 5, 32, 8, 4000, 256, 3000, 0),
    (wl.F32, 5, 32, 8, 2000, 128, 2000, 0),          # everything selected
    (wl.F32, 5, 32, 8, 1000, 64, 1000, 7),
])
def test_selections_of_many_or_wide_value_rows(dtype, B, Hq, Hkv, N, d, k, window):
    """Both sides of the rule that leaves large selections to radix select and gather."""
    q, K, V = _make(dtype, B, Hq, Hkv, N, d, seed=N + k + d)
    res = _decode(q, K, V, dtype, k, window)
    for b in sorted({0, B - 1}):
        H.check_unmargined(tuple(r[b] for r in res), q[b], K[b], V[b], dtype, k, window, f"N={N} k={k} seq {b}")


@pytest.mark.parametrize("dtype,B,Hq,Hkv,N,d,k", [
    (wl.F16, 64, 8, 8, 1024, 32, 100),               # d = 32: up to 1024 tokens
    (wl.F16, 64, 8, 8, 1025, 32, 100),
    (wl.BF16, 64, 32, 8, 3000, 32, 100),             # groups of four, 512 streams
    (wl.F16, 32, 16, 8, 3000, 64, 100),              # groups of two, one full round of streams
    (wl.F16, 33, 16, 8, 3000, 64, 100),              # a second round nearly empty
    (wl.BF16, 64, 16, 8, 1500, 256, 33),
    (wl.BF16, 32, 16, 8, 1500, 256, 33),
])
def test_both_sides_of_the_rule_for_short_sequences(dtype, B, Hq, Hkv, N, d, k):
    q, K, V = _make(dtype, B, Hq, Hkv, N, d, seed=N + k + B + d)
    res = _decode(q, K, V, dtype, k)
    for b in sorted({0, B - 1}):
        H.check_unmargined(tuple(r[b] for r in res), q[b], K[b], V[b], dtype, k, 0, f"N={N} k={k} seq {b}")
