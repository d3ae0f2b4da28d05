"""GPU parity of batches on the tile kernels in which some requests have no context at all (and so no context table)."""
import numpy as np
import pytest

from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 4, 2, 64), ("bf16", 16, 8, 256), ("f32", 4, 2, 128)])
def test_requests_without_contexts(dtype, hq, hkv, d):
    base = W.WorkloadSpec(name="tile", cfg=6, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=9,
                          chunk_lens=(40,), q_len=1, decode_steps=3, temperature=0.6, scale=0.8)
    specs = [base.replace(chunk_lens=(700, 500) if b == 2 else (33,) * (b % 2)) for b in range(6)]
    rs = [W.make_request(s, DEV, request=b) for b, s in enumerate(specs)]
    lens = [1 + b % 4 for b in range(6)]
    out, lse = H.run_decode(base, rs, lens)
    for b, r in enumerate(rs):
        ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), 1, lens[b], r.temperature, r.scale)
        H.check_close(H.f64(out[b]), ref, dtype, "request %d" % b)
        assert np.abs(H.f64(lse[b]) - ref_lse).max() <= H.lse_tol(dtype)
