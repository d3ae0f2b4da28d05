"""GPU parity of batches whose requests have contexts of very different length (every request then has splits of its own number and
length, and dense partial results): no context, one token, the edges of a 64-token unit and of a split, one long request among
short ones, more requests than one launch describes, and the batch that goes out in two launches."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import binding as B
from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _requests(dtype, hq, hkv, d, lens, q_len, own):
    spec = W.WorkloadSpec(name="uneven", cfg=7, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=9, chunk_lens=(64,),
                          q_len=q_len, decode_steps=own, temperature=0.7, scale=0.8)
    return spec, [W.make_request(spec.replace(chunk_lens=tuple(ls)), DEV, request=b) for b, ls in enumerate(lens)]


def _check(dtype, rs, out, lse, q_len, self_lens):
    for b, r in enumerate(rs):
        ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), q_len, self_lens[b], r.temperature, r.scale)
        H.check_close(H.f64(out[b]).reshape(ref.shape), ref, dtype, "request %d" % b)
        assert np.abs((H.f64(lse[b]) if q_len == 1 else H.f64(lse[b]).T.reshape(-1)) - ref_lse).max() <= H.lse_tol(dtype)


FEW = [(), (1,), (63, 1), (65,), (200, 56, 1), (700, 0, 900), (1024, 1024, 1000), (3000, 2500)]


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 32, 8, 128), ("bf16", 4, 4, 128), ("bf16", 16, 2, 128), ("bf16", 6, 3, 40), ("bf16", 4, 2, 256), ("f32", 4, 2, 64)])
@pytest.mark.parametrize("q_len", [1, 5, 40])
def test_few(dtype, hq, hkv, d, q_len):
    spec, rs = _requests(dtype, hq, hkv, d, FEW, q_len, 30)
    if q_len == 1:
        lens = [1 + 4 * b for b in range(len(rs))]
        out, lse = H.run_decode(spec, rs, lens)
    else:
        lens = [q_len + 3 * b for b in range(len(rs))]
        shape = B.make_shape(hq, hkv, d, spec.torch_dtype)
        q = torch.stack([r.q_self[n - q_len:n] for r, n in zip(rs, lens)]).contiguous()
        out, lse = torch.full_like(q, float("nan")), torch.full((len(rs), hq, q_len), float("nan"), device=DEV)
        ws = H.poisoned_workspace(B.workspace_bytes(B.APE_OP_PREFILL, shape, len(rs), q_len, 5500), DEV)
        B.attention_prefill_batch(shape, [H.make_binding_request(r, n) for r, n in zip(rs, lens)], q, out, lse, ws)
        torch.cuda.synchronize()
    _check(dtype, rs, out, lse, q_len, lens)


@pytest.mark.parametrize("batch", [16, 32, 47])
def test_many(batch):
    """32 requests on 8 KV heads have one split each in the even plan: two launches.  47: two launches by their number."""
    spec, rs = _requests("bf16", 16, 8, 128, [(37 + 91 * (b * 7 % 32),) * (1 + b % 3) for b in range(batch)], 1, 3)
    lens = [1 + b % 4 for b in range(batch)]
    out, lse = H.run_decode(spec, rs, lens)
    _check("bf16", rs, out, lse, 1, lens)
