"""The tile kernels' splits are whole stages of the form that runs (32, 64 or 128 tokens), and those of an uneven batch as short as in the even
plan: totals at the edges of stages and of splits, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import binding as B
from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [("bf16", 8, 8, 96), ("bf16", 4, 2, 256), ("f32", 4, 2, 64), ("f32", 4, 2, 128), ("f32", 2, 2, 256)]


def _spec(dtype, hq, hkv, d, lens, q_len, steps=0):
    return W.WorkloadSpec(name="units", cfg=7, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=5, chunk_lens=lens,
                          q_len=q_len, decode_steps=steps, temperature=0.8, scale=0.9)


@pytest.mark.parametrize("dtype, hq, hkv, d", SHAPES)
@pytest.mark.parametrize("total, rows", [(129, 3), (991, 3), (993, 40), (2080, 3), (2209, 70)])
def test_prefill(dtype, hq, hkv, d, total, rows):
    spec = _spec(dtype, hq, hkv, d, (total // 3, total - total // 3), rows)
    r = W.make_request(spec, DEV)
    shape = B.make_shape(hq, hkv, d, spec.torch_dtype)
    q = r.q_self[:rows].contiguous()
    out, lse = torch.full_like(q, float("nan")), torch.full((hq, rows), float("nan"), device=DEV)
    ws = H.poisoned_workspace(B.workspace_bytes(B.APE_OP_PREFILL, shape, 1, rows, total), DEV)
    B.attention_prefill(shape, H.make_binding_request(r, rows), q, out, lse, ws)
    torch.cuda.synchronize()
    ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), rows, rows, r.temperature, r.scale)
    H.check_close(H.f64(out).reshape(ref.shape), ref, dtype)
    assert np.abs(H.f64(lse).T.reshape(-1) - ref_lse).max() <= H.lse_tol(dtype)


@pytest.mark.parametrize("dtype, hq, hkv, d", SHAPES)
def test_uneven_steps(dtype, hq, hkv, d):
    lens = [(300, 97), (65,), (700, 500, 1), (1,), (257, 256)]
    spec = _spec(dtype, hq, hkv, d, (64,), 1, 8)
    rs = [W.make_request(spec.replace(chunk_lens=ls), DEV, request=b) for b, ls in enumerate(lens)]
    own = [1 + b for b in range(len(rs))]
    out, lse = H.run_decode(spec, rs, own)
    for b, r in enumerate(rs):
        ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), 1, own[b], r.temperature, r.scale)
        H.check_close(H.f64(out[b]).reshape(ref.shape), ref, dtype, "request %d" % b)
        assert np.abs(H.f64(lse[b]) - ref_lse).max() <= H.lse_tol(dtype)
