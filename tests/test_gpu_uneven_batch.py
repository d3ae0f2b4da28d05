"""GPU parity of batches whose requests have contexts of very different length (every request then has splits of its own number and
length, and dense partial results): no context, one token, the edges of a 64-token unit and of a split, one long request among
short ones, more requests than one launch describes (the last of them with a single request), and the batch that goes out in two launches."""
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


@pytest.mark.parametrize("hq, hkv, q_len", [(16, 8, 1), (16, 8, 16), (4, 4, 40), (16, 2, 40)])
def test_the_last_launch_holds_one_request(hq, hkv, q_len):
    """33 requests: a launch of 32 and one of a single long request, which is dealt out too.  Nothing is written behind the workspace."""
    spec, rs = _requests("bf16", hq, hkv, 128, [(150 + 61 * (b * 7 % 32),) for b in range(32)] + [(3000, 1096)], q_len, 3)
    n, op = len(rs), B.APE_OP_DECODE if q_len == 1 else B.APE_OP_PREFILL
    shape = B.make_shape(hq, hkv, 128, spec.torch_dtype)
    reqs = [H.make_binding_request(r, q_len + b % 4) for b, r in enumerate(rs)]
    q = torch.stack([r.q_self[b % 4:q_len + b % 4] for b, r in enumerate(rs)]).contiguous()
    size = B.workspace_bytes(op, shape, n, q_len, 4096) // 4
    ws = H.poisoned_workspace(4 * size + (32 << 20), DEV)
    ws[size:] = 7.0
    for static in ([False, True] if q_len == 1 else [False]):
        out = torch.full_like(q, float("nan"))
        lse = torch.full((n, hq) if q_len == 1 else (n, hq, q_len), float("nan"), device=DEV)
        if static:
            B.attention_decode_static(shape, reqs, q[:, 0], out[:, 0], lse)
        else:
            (B.attention_decode if q_len == 1 else B.attention_prefill_batch)(shape, reqs, q[:, 0] if q_len == 1 else q, out[:, 0] if q_len == 1 else out, lse, ws[:size])
        torch.cuda.synchronize()
        _check("bf16", rs, out, lse, q_len, [q_len + b % 4 for b in range(n)])
        assert bool((ws[size:] == 7.0).all())
