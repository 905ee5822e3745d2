"""Imports into a cache with the int8 index at the edges of the row blocks of the append kernel: rows, codes and scales as the
oracle codes them, whatever the strides of the source and the place in the cache; nothing beside them is touched."""
import numpy as np
import pytest
import torch

import helpers as H
from oracle import int8_index_ref as i8
from paper_2502_06766_amd import topk_attn as ta
from paper_2502_06766_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0) if torch.cuda.is_available() else None


@pytest.mark.parametrize("dtype,d,n,at,head_major", [
    (wl.F16, 64, 1, 0, True), (wl.BF16, 64, 127, 3, False), (wl.F16, 64, 128, 0, False), (wl.BF16, 64, 129, 1, True),
    (wl.F16, 128, 63, 0, False), (wl.BF16, 128, 64, 5, True), (wl.F16, 128, 65, 2, False), (wl.BF16, 128, 300, 0, True),
    (wl.F16, 256, 31, 0, True), (wl.BF16, 256, 32, 7, False), (wl.F16, 256, 33, 0, False),
])
def test_import_with_codes_at_the_edges_of_the_row_blocks(dtype, d, n, at, head_major):
    g = np.random.default_rng(n * d + at)
    Hkv, cap = 3, at + n + 4
    K = wl.quantize((g.standard_normal((Hkv, at + n, d)) * g.uniform(0.01, 30, (Hkv, at + n, 1))).astype(np.float32), dtype)
    V = wl.quantize(g.standard_normal((Hkv, at + n, d)).astype(np.float32), dtype)
    cache = ta.TopkAttnCache(1, 1, 3, Hkv, d, cap, 4, dtype, index_kind=ta.INDEX_INT8)
    try:
        cache.kv.fill_(0xA5)
        for a, b in ((0, at), (at, at + n)):
            if b > a:
                k, v = (H.to_torch(np.ascontiguousarray(x[:, a:b]), dtype, DEV) for x in (K, V))
                if not head_major:
                    k, v = k.permute(1, 0, 2).contiguous(), v.permute(1, 0, 2).contiguous()
                cache.append(0, 0, k, v, head_major=head_major)
        torch.cuda.synchronize()
        kv = cache.kv.cpu().numpy()
    finally:
        cache.close()
    up = lambda x: (x + 255) // 256 * 256
    rows, row_b = Hkv * cap, 2 * d
    half, codes_b = up(rows * row_b), up(rows * d)
    want_c, want_s = i8.quantize_rows_int8(wl.widen(K, dtype).astype(np.float32))
    parts = [(0, row_b, K), (half, row_b, V), (2 * half, d, want_c), (2 * half + codes_b, 4, want_s)]
    for off, width, want in parts:
        got = kv[off:off + rows * width].reshape(Hkv, cap, width)
        assert np.array_equal(got[:, :at + n].reshape(Hkv, -1), np.ascontiguousarray(want).view(np.uint8).reshape(Hkv, -1))
        assert (got[:, at + n:] == 0xA5).all()
