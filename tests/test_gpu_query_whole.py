"""GPU parity of the query calls that run without splits (one workgroup takes its rows past the contexts, then past the prefix
and the own tokens, and writes the output), on both sides of the lengths up to which they do: no context, one token, one stage
and several, requests of a batch that have contexts and that have none, scales and temperatures other than one."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import binding as B
from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _spec(dtype, hq, hkv, d, lens, q_len, prefix=9, own=0):
    return W.WorkloadSpec(name="whole", cfg=6, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=prefix,
                          chunk_lens=tuple(lens), q_len=q_len, decode_steps=own, temperature=0.6, scale=0.8)


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 8, 2, 128), ("bf16", 2, 2, 128), ("bf16", 6, 2, 40), ("bf16", 4, 2, 256),
                                               ("f32", 4, 2, 64), ("f32", 3, 1, 128), ("f32", 2, 2, 256)])
@pytest.mark.parametrize("lens, prefix", [((), 0), ((), 40), ((1,), 0), ((40, 24), 9), ((30, 0, 97, 1), 3), ((200, 56), 33), ((257,), 1), ((500, 12), 64), ((513,), 7)])
def test_lengths(dtype, hq, hkv, d, lens, prefix):
    spec = _spec(dtype, hq, hkv, d, lens, 21, prefix=prefix, own=50)
    r = W.make_request(spec, DEV)
    h = H.HostArrays(r)
    for q_len in (1, 21):
        out, lse = H.run_decode(spec, [r], [71]) if q_len == 1 else H.run_prefill(spec, r, q_len, 71)
        ref, ref_lse, _ = H.oracle_prefill(h, q_len, 71, r.temperature, r.scale)
        H.check_close(H.f64(out).reshape(-1, d), ref, dtype, "%s rows %d" % (spec, q_len))
        got = H.f64(lse).reshape(-1) if q_len == 1 else H.f64(lse).T.reshape(-1)
        assert np.abs(got - ref_lse).max() <= H.lse_tol(dtype)


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 8, 2, 128), ("bf16", 32, 8, 256), ("f32", 32, 8, 128)])
def test_batch(dtype, hq, hkv, d):
    """Also more requests than one launch describes, and steps that fill the chip (no splits whatever the length)."""
    base = _spec(dtype, hq, hkv, d, (40,), 1, own=3)
    specs = [base.replace(chunk_lens=tuple((7 + 31 * b + 17 * i) % 150 for i in range(b % 4))) for b in range(34)]
    rs = [W.make_request(s, DEV, request=b) for b, s in enumerate(specs)]
    lens = [1 + b % 4 for b in range(34)]
    out, lse = H.run_decode(base, rs, lens)
    for b, r in enumerate(rs):
        ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), 1, lens[b], r.temperature, r.scale)
        H.check_close(H.f64(out[b]), ref, dtype, "request %d" % b)
        assert np.abs(H.f64(lse[b]) - ref_lse).max() <= H.lse_tol(dtype)
