"""Keys and values at the ends of the number range, on the matrix-core kernels: keys that mask their token (a score of minus
infinity), scores of a magnitude at which fp32 resolves no single unit any more, infinite keys in heads whose width is padded, and
tokens that a row does not see and that hold no number."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _request(dtype, hq, hkv, d, lens, prefix=9, own=20, rows=21, T=0.8):
    spec = W.WorkloadSpec(name="ends", cfg=6, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=prefix,
                          chunk_lens=tuple(lens), q_len=rows, decode_steps=own, temperature=T, scale=0.9)
    return spec, W.make_request(spec, DEV)


def _lse_close(got, ref, dtype):
    assert np.all(np.abs(got - ref) <= H.lse_tol(dtype) + 1e-6 * np.abs(ref))


def _check_query(spec, r, rows=(1, 21), nodes=None):
    """Prefill, decode and tree against the oracle."""
    h, n, d = H.HostArrays(r), spec.self_len_max, spec.head_dim
    for q_len in rows:
        out, lse = H.run_decode(spec, [r], [n]) if q_len == 1 else H.run_prefill(spec, r, q_len, n)
        ref, ref_lse, _ = H.oracle_prefill(h, q_len, n, r.temperature, r.scale)
        H.check_close(H.f64(out).reshape(-1, d), ref, spec.dtype, "%s rows %d" % (spec, q_len))
        _lse_close(H.f64(lse).reshape(-1) if q_len == 1 else H.f64(lse).T.reshape(-1), ref_lse, spec.dtype)
        if nodes:
            out, lse = H.run_tree(spec, r, nodes, q_len, n)
            ref, ref_lse = H.oracle_tree(h, q_len, n, r.temperature, nodes)
            H.check_close(H.f64(out).reshape(-1, d), ref, spec.dtype, "%s tree rows %d" % (spec, q_len))
            _lse_close(H.f64(lse).T.reshape(-1), ref_lse, spec.dtype)


def _check_encode(spec, r, keep=None):
    """`keep`: the context rows that are compared (the others may hold anything)."""
    h, d, hq = H.HostArrays(r), spec.head_dim, spec.n_q_heads
    keep = np.ones(sum(r.chunk_lens), bool) if keep is None else keep
    o, lse, _, _ = H.run_encode(spec, r, with_prefix_rows=False)
    ref, ref_lse = H.oracle_encode(h)
    H.check_close(H.f64(o)[keep].reshape(-1, d), ref.reshape(-1, hq, d)[keep].reshape(-1, d), spec.dtype, "%s encode" % (spec,))
    _lse_close(H.f64(lse).T[keep], ref_lse.reshape(-1, hq)[keep], spec.dtype)


CH = 5                                                    # the channel that masks


@pytest.mark.parametrize("T", [1.0, 0.8])
@pytest.mark.parametrize("dtype, hq, hkv, d", [("f32", 3, 1, 40), ("f32", 4, 2, 64), ("f32", 4, 2, 128), ("f32", 2, 2, 256), ("bf16", 4, 2, 64), ("bf16", 2, 2, 256)])
@pytest.mark.parametrize("lens", [(40, 24), (300, 257, 65)])
def test_masked_tokens_on_the_tile_kernels(dtype, hq, hkv, d, lens, T):
    """A token whose key has the type's lowest value in one channel has the weight zero, wherever its run of 32 tokens ends."""
    spec, r = _request(dtype, hq, hkv, d, lens, T=T)
    for t in (r.q_self, r.q_ctx):
        t[..., CH] = 3.0
    low = torch.finfo(spec.torch_dtype).min
    r.k_ctx[:33, :, CH] = low                             # a whole run and a token of the next
    r.k_ctx[36::7, :, CH] = low
    r.k_self[3:6, :, CH] = low
    r.k_prefix[1:8, :, CH] = low
    _check_query(spec, r, nodes=W.tree_per_context(len(lens), 0.85))
    _check_encode(spec, r)


@pytest.mark.parametrize("low", [torch.finfo(torch.bfloat16).min, -2.0 ** 110])
@pytest.mark.parametrize("hq, hkv", [(2, 2), (8, 2), (16, 2)])
@pytest.mark.parametrize("prefix", [0, 40, 64])
def test_masked_tokens_at_the_start_of_the_encode_walk(hq, hkv, prefix, low):
    """The first block of every tile is masked (padding at the front, a masked prefix): the rows take their weights from what follows."""
    spec, r = _request("bf16", hq, hkv, 128, (12, 200, 300, 65), prefix=prefix)
    r.q_ctx[..., CH] = 3.0
    keep = np.ones(sum(r.chunk_lens), bool)
    r.k_prefix[:, :, CH] = low
    if prefix == 0:                                       # (rows that see masked tokens only have no result)
        c0 = 0
        for n in r.chunk_lens:
            r.k_ctx[c0:c0 + min(n, 32), :, CH] = low
            keep[c0:c0 + min(n, 32)] = False
            c0 += n
    _check_encode(spec, r, keep)


@pytest.mark.parametrize("q_ch, k_ch", [(1.0, -2.0 ** 105), (2.0 ** 20, 2.0 ** 20), (2.0 ** 20, -2.0 ** 20)])
@pytest.mark.parametrize("dtype, hq, hkv, d", [("f32", 3, 1, 40), ("f32", 4, 2, 64), ("f32", 2, 2, 256), ("bf16", 4, 2, 64), ("bf16", 2, 2, 256)])
@pytest.mark.parametrize("lens", [(40, 24), (300, 257, 65)])
def test_scores_of_any_magnitude_on_the_tile_kernels(dtype, hq, hkv, d, lens, q_ch, k_ch):
    """All of a row's scores far from zero and from each other, as products that fp32 holds exactly up to the scale (q has one
    channel): one token takes all of the weight.  (Not under a tree, whose merge works with differences of log-weights.)"""
    spec, r = _request(dtype, hq, hkv, d, lens)
    for t in (r.q_self, r.q_ctx):
        t[:] = 0.0
        t[..., CH] = q_ch
    for i, t in enumerate((r.k_prefix, r.k_ctx, r.k_self)):
        at = torch.arange(t.shape[0], device=DEV)         # 8 bits of mantissa: no two alike
        t[..., CH] = (k_ch * (1.0 + at * 37 % 128 / 128.0) * 2.0 ** (at // 128 - (1, 0, 2)[i])).to(t.dtype)[:, None]
    _check_query(spec, r)
    _check_encode(spec, r)
