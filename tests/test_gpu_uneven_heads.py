"""GPU parity of uneven decode steps on many KV heads of 128: one launch with two splits for each request, two launches of half the requests
each, the even plan where there is nothing to deal out, and tile-kernel batches whose splits are whole stages."""
import numpy as np
import pytest

from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype, hq, hkv, d, batch, lens", [
    ("bf16", 16, 16, 128, 16, lambda b: (90 + 300 * (b * 7 % 16),)),                 # one split each in the even plan: two launches
    ("bf16", 16, 16, 128, 24, lambda b: (1 + 200 * (b * 5 % 24), 65)),               # one launch, two splits a request
    ("bf16", 32, 32, 128, 12, lambda b: (64 * b, 300 * (b % 2), 129)),
    ("bf16", 32, 32, 128, 40, lambda b: (37 + 91 * (b * 7 % 32),)),                  # short: the even plan, two launches by the requests' number
    ("bf16", 8, 8, 128, 4, lambda b: (512, 256, 1024, 256)[b:b + 1]),                # the even plan's own splits
    ("bf16", 8, 8, 96, 10, lambda b: (203,) * (1 + 2 * b)),
    ("bf16", 6, 2, 40, 9, lambda b: (128 + b, 511)[b % 2:]),
    ("f32", 4, 2, 64, 7, lambda b: (129 * (b + 1),) if b != 3 else ())])
def test_steps(dtype, hq, hkv, d, batch, lens):
    spec = W.WorkloadSpec(name="heads", cfg=7, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=9, chunk_lens=(64,),
                          q_len=1, decode_steps=5, temperature=0.7, scale=0.8)
    rs = [W.make_request(spec.replace(chunk_lens=tuple(lens(b))), DEV, request=b) for b in range(batch)]
    own = [1 + b % 5 for b in range(batch)]
    out, lse = H.run_decode(spec, rs, own)
    for b, r in enumerate(rs):
        ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), 1, own[b], r.temperature, r.scale)
        H.check_close(H.f64(out[b]).reshape(ref.shape), ref, dtype, "request %d" % b)
        assert np.abs(H.f64(lse[b]) - ref_lse).max() <= H.lse_tol(dtype)
