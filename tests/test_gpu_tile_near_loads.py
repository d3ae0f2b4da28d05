"""The tile kernels load a stage that lies within one segment with one base and 32-bit offsets per lane, and any other row by row.  The same
tokens in one context (stages of both kinds only at its end) and cut so that contexts end inside, at and next to the ends of stages are
the same stages of the same numbers: the outputs are the same bits, and those of the oracle."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import binding as B
from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CUTS = [(32, 608), (31, 1, 32, 576), (33, 95, 128, 384), (64, 1, 63, 127, 129, 256), (160, 0, 160, 320), tuple([20] * 32)]


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 4, 2, 64), ("bf16", 6, 2, 40), ("bf16", 8, 8, 96), ("bf16", 12, 2, 128), ("bf16", 4, 2, 256), ("bf16", 4, 2, 200),
                                               ("f32", 4, 2, 64), ("f32", 6, 2, 40), ("f32", 4, 2, 128), ("f32", 4, 2, 256), ("f32", 4, 2, 136)])
@pytest.mark.parametrize("rows", [7, 45])
def test_cuts(dtype, hq, hkv, d, rows):
    spec = W.WorkloadSpec(name="near", cfg=7, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=32, chunk_lens=(640,),
                          q_len=rows, decode_steps=0, temperature=0.8, scale=0.9)
    r = W.make_request(spec, DEV)
    shape = B.make_shape(hq, hkv, d, spec.torch_dtype)
    k, v = (x[0] for x in r.chunk_views())
    q = r.q_self[:rows].contiguous()

    def prefill(lens):
        at = np.cumsum([0, *lens])
        ks, vs = ([x[a:b].clone() for a, b in zip(at[:-1], at[1:])] for x in (k, v))
        req = B.Request(r.k_prefix, r.v_prefix, ks, vs, r.k_self, r.v_self, rows, r.temperature, r.scale)
        out, lse = torch.full_like(q, float("nan")), torch.full((hq, rows), float("nan"), device=DEV)
        ws = H.poisoned_workspace(B.workspace_bytes(B.APE_OP_PREFILL, shape, 1, rows, 640), DEV)
        B.attention_prefill(shape, req, q, out, lse, ws)
        torch.cuda.synchronize()
        return out, lse

    out, lse = prefill((640,))
    ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), rows, rows, r.temperature, r.scale)
    H.check_close(H.f64(out).reshape(ref.shape), ref, dtype)
    assert np.abs(H.f64(lse).T.reshape(-1) - ref_lse).max() <= H.lse_tol(dtype)
    for lens in CUTS:
        other, other_lse = prefill(lens)
        assert torch.equal(other, out) and torch.equal(other_lse, lse), lens
