"""GPU parity of the tile kernels (every head shape beside the flash kernels': bf16 and fp32, any
head_dim, any number of query heads per KV head) where they can go wrong: head_dims at the edges of the
padded widths, row counts at the edges of the row tiles, contexts that begin inside a stage of tokens
(also several of them, and empty ones), streams shorter and longer than the ring."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _spec(dtype, hq, hkv, d, lens, q_len, prefix=9, own=0):
    return W.WorkloadSpec(name="tile", cfg=6, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=prefix,
                          chunk_lens=tuple(lens), q_len=q_len, decode_steps=own, temperature=0.8, scale=0.9)


def _check(spec, nodes=None):
    r = W.make_request(spec, DEV)
    h = H.HostArrays(r)
    n, d = spec.self_len_max, spec.head_dim
    tol = H.lse_tol(spec.dtype)
    for q_len in sorted({1, spec.q_len}):
        out, lse = H.run_decode(spec, [r], [n]) if q_len == 1 else H.run_prefill(spec, r, q_len, n)
        ref, ref_lse, _ = H.oracle_prefill(h, q_len, n, r.temperature, r.scale)
        H.check_close(H.f64(out).reshape(-1, d), ref, spec.dtype, "%s rows %d" % (spec, q_len))
        got = H.f64(lse).reshape(-1) if q_len == 1 else H.f64(lse).T.reshape(-1)
        assert np.abs(got - ref_lse).max() <= tol
        if nodes:
            out, lse = H.run_tree(spec, r, nodes, q_len, n)
            ref, ref_lse = H.oracle_tree(h, q_len, n, r.temperature, nodes)
            H.check_close(H.f64(out).reshape(-1, d), ref, spec.dtype, "%s tree rows %d" % (spec, q_len))
            assert np.abs(H.f64(lse).T.reshape(-1) - ref_lse).max() <= tol
    o_ctx, lse_ctx, o_p, lse_p = H.run_encode(spec, r)
    ref, ref_lse = H.oracle_encode(h)
    H.check_close(H.f64(o_ctx).reshape(-1, d), ref, spec.dtype, "%s encode" % (spec,))
    assert np.abs(H.f64(lse_ctx).T.reshape(-1) - ref_lse).max() <= tol
    if o_p is not None:
        refp, _ = H.oracle_encode_prefix(h)
        H.check_close(H.f64(o_p).reshape(-1, d), refp, spec.dtype, "%s prefix rows" % (spec,))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hq, hkv, d", [(2, 2, 8), (3, 1, 40), (4, 2, 64), (6, 2, 72), (5, 1, 128), (12, 1, 136), (16, 8, 256)])
def test_head_shapes(dtype, hq, hkv, d):
    _check(_spec(dtype, hq, hkv, d, (33, 100, 1, 64, 257), 20, own=3), W.tree_per_context(5, 0.85))


@pytest.mark.parametrize("dtype, d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 256)])
@pytest.mark.parametrize("q_len", [31, 32, 33, 64, 65, 128, 129, 300])
def test_row_tiles(dtype, d, q_len):
    _check(_spec(dtype, 2, 2, d, (90, 40), q_len))


@pytest.mark.parametrize("dtype, hq, hkv, d", [("f32", 3, 1, 64), ("f32", 2, 1, 256), ("bf16", 6, 2, 64), ("bf16", 2, 2, 256), ("bf16", 6, 2, 128)])
@pytest.mark.parametrize("lens, prefix", [
    ((1,) * 200, 0),                                      # dozens of contexts inside one stage
    ((7, 0, 0, 30, 0, 3, 150, 0, 1, 1, 1, 29, 31, 32, 33, 0), 5),   # empty ones between, at the start and at the end of stages
    ((0, 0, 5, 0), 1),                                    # a stream shorter than one run of tokens
    ((700, 1, 650), 64),                                  # longer than the ring, boundaries deep inside
    ((), 33),                                             # no context at all
])
def test_contexts_inside_stages(dtype, hq, hkv, d, lens, prefix):
    spec = _spec(dtype, hq, hkv, d, lens, 40, prefix=prefix, own=70)
    if lens:
        _check(spec, W.tree_grouped(len(lens), 3, 0.95, 0.85))
    r = W.make_request(spec, DEV)                         # every context in a buffer of its own
    h = H.HostArrays(r)
    out, _ = H.run_prefill(spec, r, 40, 110, req=H.make_binding_request(r, 110, separate_buffers=True))
    ref, _, _ = H.oracle_prefill(h, 40, 110, r.temperature, r.scale)
    H.check_close(H.f64(out).reshape(-1, d), ref, dtype, "separate buffers")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_late_outliers_move_the_softmax_reference(dtype):
    """Scores that tower over everything before them, deep inside a stream: the accumulators are rescaled there.
    fp32: a score of magnitude 100 carries a rounding error of about 100 * 6e-8 * sqrt(64 / 4 terms a chain), i.e. a few
    1e-5 of its probability where two such scores compete; one towers alone here, so the plain bound holds."""
    spec = _spec(dtype, 6, 2, 64, (300, 500), 30, own=5)
    r = W.make_request(spec, DEV)
    for hk in range(2):
        r.k_ctx[250 + hk, hk] = 8.0 * r.q_self[10 + hk, 3 * hk]
        r.k_ctx[640, hk] = 9.0 * r.q_self[20, 3 * hk + 2]
        r.k_ctx[200, hk] = 8.0 * r.q_ctx[290, 3 * hk + 1]
    h = H.HostArrays(r)
    out, _ = H.run_prefill(spec, r, 30, 35)
    ref, _, _ = H.oracle_prefill(h, 30, 35, r.temperature, r.scale)
    H.check_close(H.f64(out).reshape(-1, 64), ref, dtype, "outliers")
    o_ctx, _, _, _ = H.run_encode(spec, r)
    ref, _ = H.oracle_encode(h)
    H.check_close(H.f64(o_ctx).reshape(-1, 64), ref, dtype, "outliers encode")
    assert (r.q_self[10].float()[0] * r.k_ctx[250, 0].float()).sum().item() / 8.0 / 0.8 > 40.0


def test_batch_of_mixed_requests():
    """More requests than one launch describes, of different lengths: trailing splits of the short ones stay untouched."""
    base = _spec("bf16", 6, 2, 96, (64,), 1, own=4)
    specs = [base.replace(chunk_lens=tuple(20 + (13 * b + 31 * i) % 90 for i in range(1 + b % 9))) for b in range(35)]
    rs = [W.make_request(s, DEV, request=b) for b, s in enumerate(specs)]
    lens = [1 + b % 5 for b in range(35)]
    out, lse = H.run_decode(base, rs, lens)
    for b, r in enumerate(rs):
        ref, ref_lse, _ = H.oracle_prefill(H.HostArrays(r), 1, lens[b], r.temperature, r.scale)
        H.check_close(H.f64(out[b]), ref, "bf16", "request %d" % b)
        assert np.abs(H.f64(lse[b]) - ref_lse).max() <= H.lse_tol("bf16")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_uneven_contexts_of_wide_heads(dtype):
    """One long context among thousands of one token: the grid has room for tiles of 128 rows only.  Against the vector-ALU kernels."""
    spec = _spec(dtype, 16, 2, 136, (3,) + (1,) * 16400 + (4090,), 1, prefix=5)
    r = W.make_request(spec, DEV)
    o, lse, _, _ = H.run_encode(spec, r, with_prefix_rows=False)
    ref, ref_lse, _, _ = H.run_encode(spec, r, generic=True, with_prefix_rows=False)
    H.check_close(H.f64(o), H.f64(ref), dtype, "uneven contexts")
    assert (lse - ref_lse).abs().max().item() <= H.lse_tol(dtype)
