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


@pytest.mark.parametrize("dtype, hq, hkv, d", [("f32", 3, 1, 40), ("f32", 6, 2, 72), ("f32", 2, 2, 136), ("bf16", 6, 2, 40), ("bf16", 8, 8, 96), ("bf16", 2, 2, 200)])
@pytest.mark.parametrize("lens", [(40, 24), (300, 257, 65)])
def test_infinite_keys_in_padded_heads(dtype, hq, hkv, d, lens):
    """A key of minus infinity in one of its first channels, which is what the padding repeated."""
    spec, r = _request(dtype, hq, hkv, d, lens)
    for t in (r.q_self, r.q_ctx):
        t[..., 0] = 3.0
    r.k_ctx[2::5, :, 0] = -float("inf")
    r.k_self[2, :, 0] = -float("inf")
    _check_query(spec, r, nodes=W.tree_per_context(len(lens), 0.85))
    _check_encode(spec, r)


@pytest.mark.parametrize("what", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("dtype, hq, hkv, d", [("f32", 3, 1, 40), ("f32", 4, 2, 64), ("f32", 8, 4, 128), ("f32", 2, 2, 256), ("bf16", 4, 2, 64), ("bf16", 6, 2, 96), ("bf16", 4, 2, 256)])
@pytest.mark.parametrize("lens", [(70, 40), (300, 90), (130,) * 40])
def test_hidden_tokens_leave_no_trace_on_the_tile_kernels(dtype, hq, hkv, d, lens, what):
    """Tokens that hold no numbers, from some place on in a context and in the own tokens: the rows in front of them are those of a
    request without them."""
    spec, r = _request(dtype, hq, hkv, d, lens, prefix=5, own=7, rows=80)
    n = spec.self_len_max
    h = H.HostArrays(r)
    at = [17, 39, 5, 33][:len(lens)] + [50] * (len(lens) - 4)     # first row of each context that sees one
    keep, c0 = np.ones(sum(lens), bool), 0
    for a, ln in zip(at, lens):
        keep[c0 + a:c0 + ln] = False
        c0 += ln
    refs = H.oracle_encode(h) if len(lens) < 10 else H.run_encode(spec, r, with_prefix_rows=False)[:2]
    first = 7 + 45                                            # ... and first own token
    dirty = [t.clone() for t in (r.k_ctx, r.v_ctx, r.k_self, r.v_self)]
    for t in dirty[:2]:
        t[torch.from_numpy(~keep).to(DEV)] = what
    for t in dirty[2:]:
        t[first:] = what
    clean = r.k_self, r.v_self, r.k_ctx, r.v_ctx
    r.k_ctx, r.v_ctx = dirty[:2]
    o, lse, _, _ = H.run_encode(spec, r, with_prefix_rows=False)
    r.k_ctx, r.v_ctx = clean[2:]
    if len(lens) < 10:
        ref, ref_lse = refs[0].reshape(-1, hq, d), refs[1].reshape(-1, hq)
    else:
        ref, ref_lse = H.f64(refs[0]), H.f64(refs[1]).T
    H.check_close(H.f64(o)[keep].reshape(-1, d), ref[keep].reshape(-1, d), dtype, "encode")
    _lse_close(H.f64(lse).T[keep], ref_lse[keep], dtype)
    assert not torch.isfinite(o.float())[torch.from_numpy(~keep).to(DEV)].any()
    nodes = W.tree_per_context(len(lens), 0.85)
    for rows in (80, 60):
        ref, ref_lse, _ = H.oracle_prefill(h, rows, n, r.temperature, r.scale)
        tref, tref_lse = H.oracle_tree(h, rows, n, r.temperature, nodes)
        r.k_self, r.v_self = dirty[2:]
        got = H.run_prefill(spec, r, rows, n), H.run_tree(spec, r, nodes, rows, n)
        r.k_self, r.v_self = clean[:2]
        seen = first - (n - rows)                             # rows in front of the first such token
        for (o, lse), want, want_lse in zip(got, (ref, tref), (ref_lse, tref_lse)):
            H.check_close(H.f64(o)[:seen].reshape(-1, d), want.reshape(rows, hq, d)[:seen].reshape(-1, d), dtype, "%d rows" % rows)
            _lse_close(H.f64(lse).T[:seen], want_lse.reshape(rows, hq)[:seen], dtype)
            assert not torch.isfinite(o.float())[seen:].any()
