"""GPU parity of the tile kernels' encode over the ways its tiles are dealt out: one group of contexts, a group that ends by its number
of contexts (64) or by its bytes, contexts without tokens at the ends of groups, more groups than one call lists, one context."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype, hq, hkv, d, lens, prefix", [
    ("f32", 6, 2, 40, [1], 0), ("f32", 4, 2, 64, [33, 1, 64, 0, 65], 7),
    ("f32", 3, 1, 40, [(7 * i) % 40 for i in range(131)], 5),                        # groups of 64, 64 and 3 contexts
    ("bf16", 2, 1, 256, [600, 424, 0, 1, 300, 723, 1, 0], 9),                        # 1024 tokens of 256 dims: 1 MB
    ("bf16", 2, 1, 256, [1024, 1, 1023, 0, 1100], 3),
    ("bf16", 8, 8, 96, [0, 0, 130, 5, 0, 128], 32),
    ("bf16", 6, 2, 40, [(5 * i) % 4 for i in range(64 * 31 + 7)], 3),                # 32 groups: by contexts, as larger calls
    ("f32", 4, 1, 128, [(i * 37) % 400 for i in range(60)], 16)])
def test_order(dtype, hq, hkv, d, lens, prefix):
    spec = W.WorkloadSpec(name="order", cfg=8, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=prefix, chunk_lens=tuple(lens),
                          q_len=1, decode_steps=0)
    r = W.make_request(spec, DEV)
    out, lse, o_p, lse_p = H.run_encode(spec, r)
    h = H.HostArrays(r)
    ref, ref_lse = H.oracle_encode(h)
    H.check_close(H.f64(out).reshape(ref.shape), ref, dtype, "rows")
    assert np.abs(H.f64(lse).T.reshape(-1) - ref_lse.reshape(-1)).max() <= H.lse_tol(dtype)
    if prefix:
        ref, ref_lse = H.oracle_encode_prefix(h)
        H.check_close(H.f64(o_p).reshape(ref.shape), ref, dtype, "prefix rows")
