"""Query calls of the tile kernels whose splits' teams (split, KV head) are no multiple of the eight XCDs: the prefix and own tokens' teams are
numbered on from them, in one request, in a batch and in an uneven batch."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import binding as B
from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype, hq, hkv, d", [("f32", 2, 2, 256), ("f32", 3, 3, 64), ("bf16", 6, 1, 128), ("bf16", 10, 5, 40)])
@pytest.mark.parametrize("rows", [3, 70])
@pytest.mark.parametrize("lens", [((700,),), ((1500,),), ((513, 512), (1025,), (1000,)), ((40, 300), (1300, 100), (), (2000,))])
def test_teams(dtype, hq, hkv, d, rows, lens):
    spec = W.WorkloadSpec(name="teams", cfg=7, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=5, chunk_lens=(64,),
                          q_len=rows, decode_steps=0, temperature=0.8, scale=0.9)
    rs = [W.make_request(spec.replace(chunk_lens=ls), DEV, request=b) for b, ls in enumerate(lens)]
    shape = B.make_shape(hq, hkv, d, spec.torch_dtype)
    q = torch.stack([r.q_self[:rows] for r in rs]).contiguous()
    out, lse = torch.full_like(q, float("nan")), torch.full((len(rs), hq, rows), float("nan"), device=DEV)
    ws = H.poisoned_workspace(B.workspace_bytes(B.APE_OP_PREFILL, shape, len(rs), rows, max(map(sum, lens))), DEV)
    B.attention_prefill_batch(shape, [H.make_binding_request(r, rows) for r in rs], q, out, lse, ws)
    torch.cuda.synchronize()
    for b, r in enumerate(rs):
        ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), rows, rows, r.temperature, r.scale)
        H.check_close(H.f64(out[b]).reshape(ref.shape), ref, dtype, "request %d" % b)
        assert np.abs(H.f64(lse[b]).T.reshape(-1) - ref_lse).max() <= H.lse_tol(dtype)
