"""Selection of the one launch over short sequences where it can go wrong: slots only some lanes have, bins that crowd and are
split again, scores that are all equal or spread over almost all of fp32.  All elements of q and K are small multiples of a power of two,
so the scores are exact in fp32 and the selection has to equal the oracle's, ties to the lower position."""
import numpy as np
import pytest
import torch

import helpers as H
from oracle import c_oracle
from paper_2502_06766_amd import topk_attn as ta
from paper_2502_06766_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0) if torch.cuda.is_available() else None


@pytest.mark.parametrize("dtype,lens,Hq,Hkv,d,k,kind", [
    (wl.F16, [1, 63, 64, 65, 500], 8, 2, 64, 70, "plain"),
    (wl.BF16, [512, 511, 449, 20], 4, 4, 128, 300, "plain"),
    (wl.F16, [512, 300], 6, 2, 32, 16, "equal"),
    (wl.BF16, [500, 512, 100], 8, 2, 256, 65, "few values"),           # hundreds of ties in the k-th score's bin
    (wl.F16, [512, 65], 4, 1, 64, 40, "outlier"),                      # all others in one bin
    (wl.F16, [4096, 4095, 2048, 2500] * 32, 8, 2, 64, 256, "plain"),
    (wl.BF16, [4000, 3001] * 64, 8, 2, 128, 100, "few values"),
    (wl.F16, [2047, 1025] * 64, 8, 2, 64, 512, "outlier"),
])
def test_short_sequences(dtype, lens, Hq, Hkv, d, k, kind):
    g = np.random.default_rng(len(lens) * 1000 + k)
    B, n_max = len(lens), max(lens)
    shown = [b for b in range(B) if b < 4 or b >= B - 2]               # judged by the oracle (the rest repeats their lengths)
    hi = 1 if kind == "few values" else 8
    q = wl.quantize(g.integers(-3, 4, (B, Hq, d)).astype(np.float32), dtype)
    cache = ta.TopkAttnCache(1, B, Hq, Hkv, d, n_max, k, dtype)
    try:
        data = {}
        for b, n in enumerate(lens):
            K = g.integers(-hi, hi + 1, (Hkv, n, d)).astype(np.float32)
            if kind == "equal":
                K[:] = K[:, :1]
            if kind == "few values":
                K[:, :, 2:] = 0
            if kind == "outlier" and n > 8:
                K[:, n // 2] *= 256
                K[:, n // 3] *= -256
            V = g.standard_normal((Hkv, n, d)).astype(np.float32)
            K, V = wl.quantize(K, dtype), wl.quantize(V, dtype)
            cache.append(0, b, H.to_torch(K, dtype, DEV), H.to_torch(V, dtype, DEV), head_major=True)
            if b in shown:
                data[b] = (K, V)
        qd = H.to_torch(q, dtype, DEV)
        res = cache.decode(0, qd, k)
        again = cache.decode(0, qd, k)
        torch.cuda.synchronize()
        for x, y in zip(res, again):
            assert torch.equal(x, y)
        for b in shown:
            K, V = data[b]
            ref = c_oracle.topk_attention(q[b], K, V, dtype, k)
            H.check_against_oracle(*(r[b].cpu().numpy() for r in res), ref, np.full(Hq, 1e-30), min(k, lens[b]), H.out_tolerance(dtype),
                                   float(np.abs(wl.widen(V, dtype)).max()), f"{kind} seq {b} n={lens[b]}")
    finally:
        cache.close()
