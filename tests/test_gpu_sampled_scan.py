"""The filter scan that works its heads' thresholds out itself, at the ends of the range of sample sizes it takes over, against the
oracle: groups of one to four heads, ragged batches (a sequence may have a smaller sample, too few tokens to filter, or
nothing to search), and the chip-wide tail behind it, which reads the bins the scan leaves."""
import numpy as np
import pytest
import torch

import helpers as H
from paper_2502_06766_amd import topk_attn as ta
from paper_2502_06766_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0) if torch.cuda.is_available() else None


@pytest.mark.parametrize("dtype,Hq,Hkv,d,lens,k,window", [
    (wl.F16, 4, 1, 64, [135167], 300, 0),                    # the largest sample a wave takes (2048)
    (wl.F16, 4, 1, 64, [135168], 300, 0),                    # one stratum more: a launch of its own
    (wl.BF16, 2, 2, 128, [65536 + 63], 40, 0),               # groups of one, the smallest sample (1024)
    (wl.F16, 6, 2, 256, [30011], 500, 0),                    # groups of three, one tile buffer per wave
    (wl.BF16, 4, 2, 32, [40000], 2000, 0),
    (wl.F16, 8, 2, 64, [70000, 100, 40000, 255, 64], 300, 64),   # ragged: not filterable, inside the window
    (wl.BF16, 8, 2, 128, [60000, 60000], 9000, 0),           # dense selections: the chip-wide tail follows
])
def test_thresholds_worked_out_by_the_scan(dtype, Hq, Hkv, d, lens, k, window):
    g = np.random.default_rng(sum(lens) + k)
    B = len(lens)
    q = wl.quantize(g.standard_normal((B, Hq, d)).astype(np.float32), dtype)
    K = [wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), dtype) for n in lens]
    V = [wl.quantize(g.standard_normal((Hkv, n, d)).astype(np.float32), dtype) for n in lens]
    cache = ta.TopkAttnCache(1, B, Hq, Hkv, d, max(lens), k, dtype, max_window=window)
    try:
        for b in range(B):
            cache.append(0, b, H.to_torch(K[b], dtype, DEV), H.to_torch(V[b], dtype, DEV), head_major=True)
        cache.set_path(ta.PATH_FILTER)
        qd = H.to_torch(q, dtype, DEV)
        res = cache.decode(0, qd, k, window=window)
        again = cache.decode(0, qd, k, window=window)
        torch.cuda.synchronize()
        assert cache.last_fallbacks() == 0
        for a, b in zip(res, again):
            assert torch.equal(a, b)
        for b in range(B):
            H.check_unmargined(tuple(t[b].cpu().numpy() for t in res), q[b], K[b], V[b], dtype, k, window, f"seq {b}")
    finally:
        cache.close()


@pytest.mark.parametrize("dtype,Hq,Hkv,d,lens,k,window", [
    (wl.F16, 16, 4, 64, [135167], 300, 0),                   # four key streams, the fewest that do without a launch; the largest sample
    (wl.F16, 16, 4, 64, [135168], 300, 0),
    (wl.F16, 12, 3, 64, [135167], 300, 0),                   # three
    (wl.BF16, 4, 4, 128, [65536 + 63], 40, 0),               # groups of one
    (wl.F16, 12, 4, 128, [30011], 500, 0),                   # groups of three
    (wl.F16, 12, 4, 256, [30011], 500, 0),                   # one tile buffer per wave: a launch of its own
    (wl.BF16, 8, 4, 32, [40000], 2000, 0),
    (wl.BF16, 16, 4, 128, [60000], 9000, 0),                 # the chip-wide tail follows
])
def test_the_same_with_more_key_streams(dtype, Hq, Hkv, d, lens, k, window):
    test_thresholds_worked_out_by_the_scan(dtype, Hq, Hkv, d, lens, k, window)
