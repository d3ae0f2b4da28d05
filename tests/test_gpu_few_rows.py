"""GPU parity of the few-row kernels (tiles of 16 (token, head) rows per KV head) against the oracle: head_dims that fill LDS rows and that do not,
blocks of 32 tokens that end with a context and that hold several, more contexts than the lanes hold at once, both sides of the lengths up to which a
call runs without splits, batches, the tree, tokens that a row does not see."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import binding as B
from paper_2502_05431_amd import workloads as W

import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPES = [("bf16", 8, 2, 128), ("bf16", 16, 1, 128), ("bf16", 3, 3, 128), ("bf16", 16, 8, 256), ("bf16", 5, 1, 200), ("bf16", 8, 2, 64), ("bf16", 6, 2, 40),
          ("bf16", 8, 8, 96), ("bf16", 7, 1, 8), ("f32", 8, 2, 128), ("f32", 5, 1, 72), ("f32", 4, 2, 64), ("f32", 16, 1, 40)]


def _spec(dtype, hq, hkv, d, lens, q_len, prefix, own):
    return W.WorkloadSpec(name="few", cfg=6, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=prefix,
                          chunk_lens=tuple(lens), q_len=q_len, decode_steps=own, temperature=0.6, scale=0.8)


def _check(spec, r, q_len, self_len, out, lse, h=None):
    ref, ref_lse, _ = H.oracle_prefill(h or H.HostArrays(r), q_len, self_len, r.temperature, r.scale)
    H.check_close(H.f64(out).reshape(-1, spec.head_dim), ref, spec.dtype, "%s rows %d" % (spec, q_len))
    got = H.f64(lse).reshape(-1) if lse.shape[0] != spec.n_q_heads or lse.dim() == 1 else H.f64(lse).T.reshape(-1)
    assert np.abs(got - ref_lse).max() <= H.lse_tol(spec.dtype)


@pytest.mark.parametrize("dtype, hq, hkv, d", SHAPES)
@pytest.mark.parametrize("lens, prefix, own", [
    ((31,), 0, 0), ((32,), 32, 31), ((33, 95), 7, 33), ([2] * 70 + [0] * 3 + [1, 61], 1, 5), ([0, 40, 0, 25, 64] * 26 + [3], 40, 300),
    ((384,), 0, 1), ((385,), 0, 1), ((300, 213), 5, 60), ((1000, 1, 1047), 64, 100), ([128] * 3, 600, 900)])
def test_streams(dtype, hq, hkv, d, lens, prefix, own):
    rows = max(1, 16 // (hq // hkv))
    spec = _spec(dtype, hq, hkv, d, lens, rows, prefix, own)
    r = W.make_request(spec, DEV)
    h = H.HostArrays(r)
    req = H.make_binding_request(r, own + rows, separate_buffers=True)
    for q_len in {1, rows}:
        out, lse = H.run_decode(spec, [r], [own + rows], reqs=[req]) if q_len == 1 else H.run_prefill(spec, r, q_len, own + rows, req=req)
        _check(spec, r, q_len, own + rows, out, lse[0] if q_len == 1 else lse, h)


@pytest.mark.parametrize("dtype, hq, hkv, d, n, ctx", [
    ("bf16", 8, 2, 128, 35, 300), ("bf16", 32, 8, 128, 17, 900), ("bf16", 8, 2, 128, 9, 900), ("bf16", 16, 8, 256, 3, 500), ("bf16", 8, 8, 96, 5, 700),
    ("bf16", 8, 2, 64, 20, 1500), ("f32", 8, 2, 128, 34, 110), ("f32", 4, 2, 64, 5, 900), ("f32", 16, 8, 128, 17, 400)])
def test_batches(dtype, hq, hkv, d, n, ctx):
    specs = [_spec(dtype, hq, hkv, d, (ctx - 3 * b - 40, 40 + 2 * b), 1, 11, 40) for b in range(n)]
    rs = [W.make_request(s, DEV, request=b) for b, s in enumerate(specs)]
    lens = [1 + (7 * b) % 40 for b in range(n)]
    out, lse = H.run_decode(specs[0], rs, lens)
    for b in range(n):
        _check(specs[b], rs[b], 1, lens[b], out[b], lse[b])


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 8, 2, 128), ("bf16", 4, 2, 256), ("bf16", 6, 2, 40), ("f32", 4, 2, 64), ("f32", 8, 2, 128)])
@pytest.mark.parametrize("nodes", ["per_context", "grouped"])
def test_tree(dtype, hq, hkv, d, nodes):
    lens = [50, 1, 128, 33, 300, 64, 2, 95]
    tree = W.tree_per_context(len(lens), 0.85) if nodes == "per_context" else W.tree_grouped(len(lens), 3, 0.9, 0.85)
    spec = _spec(dtype, hq, hkv, d, lens, 2, 20, 30)
    r = W.make_request(spec, DEV)
    h = H.HostArrays(r)
    for q_len in (1, 2):
        out, lse = H.run_tree(spec, r, tree, q_len, 32)
        ref, ref_lse = H.oracle_tree(h, q_len, 32, r.temperature, tree)
        H.check_close(H.f64(out).reshape(-1, d), ref, dtype, "tree")
        assert np.abs(H.f64(lse).T.reshape(-1) - ref_lse).max() <= H.lse_tol(dtype)


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 8, 2, 128), ("bf16", 4, 2, 256), ("bf16", 6, 2, 40), ("f32", 4, 2, 64), ("f32", 5, 1, 72)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("ctx", [100, 900])
def test_a_token_that_a_row_does_not_see(dtype, hq, hkv, d, value, ctx):
    """Rows in front of a token that holds no number keep their results; the last row sees it."""
    spec = _spec(dtype, hq, hkv, d, (ctx,), 3, 5, 20)
    r = W.make_request(spec, DEV)
    h = H.HostArrays(r)
    ref, _, _ = H.oracle_prefill(h, 3, 23, r.temperature, r.scale)
    r.v_self[22] = value
    out, _ = H.run_prefill(spec, r, 3, 23)
    H.check_close(H.f64(out[:2]).reshape(-1, d), ref[:2 * hq], dtype, "rows in front of it")
    assert not torch.isfinite(out[2].float()).any()


@pytest.mark.parametrize("dtype, hq, hkv, d, rows, lens", [
    ("bf16", 8, 2, 128, 5, (300, 468)), ("bf16", 32, 8, 128, 128, (33, 70)), ("bf16", 3, 1, 128, 170, (400,)), ("bf16", 4, 2, 256, 40, (250, 6)), ("bf16", 8, 2, 64, 33, (1000, 24)),
    ("f32", 4, 2, 64, 16, (32,) * 4), ("f32", 8, 2, 128, 21, (200, 56)), ("f32", 3, 3, 40, 100, (100,)), ("bf16", 6, 2, 40, 7, ()),
    ("bf16", 8, 2, 128, 21, (900, 1, 800)), ("bf16", 32, 8, 128, 32, (2048,)), ("bf16", 3, 1, 200, 100, (310, 500)), ("f32", 8, 2, 128, 9, (700, 1400)), ("f32", 6, 2, 40, 33, (1500,)),
    ("bf16", 255, 1, 8, 2, (40,)), ("bf16", 171, 1, 8, 2, (33, 9)), ("f32", 127, 1, 8, 4, (40,)), ("bf16", 512, 1, 8, 1, (70,))])
def test_tiles_of_rows(dtype, hq, hkv, d, rows, lens):
    spec = _spec(dtype, hq, hkv, d, lens, rows, 9, 40)
    for batch in (1, 2):
        rs = [W.make_request(spec, DEV, request=b) for b in range(batch)]
        if batch == 1:
            out, lse = H.run_prefill(spec, rs[0], rows, 40 + rows)
            _check(spec, rs[0], rows, 40 + rows, out, lse)
            continue
        shape = B.make_shape(hq, hkv, d, spec.torch_dtype)
        q = torch.stack([r.q_self[40:40 + rows] for r in rs]).contiguous()
        out, lse = torch.full_like(q, float("nan")), torch.full((batch, hq, rows), float("nan"), device=DEV)
        ws = H.poisoned_workspace(B.workspace_bytes(B.APE_OP_PREFILL, shape, batch, rows, sum(lens)), DEV)
        B.attention_prefill_batch(shape, [H.make_binding_request(r, 40 + rows) for r in rs], q, out, lse, ws)
        torch.cuda.synchronize()
        for b in range(batch):
            _check(spec, rs[b], rows, 40 + rows, out[b], lse[b])


@pytest.mark.parametrize("dtype, hq, hkv, d, n, ctx, own", [
    ("bf16", 32, 8, 128, 8, 900, 40), ("bf16", 32, 8, 128, 9, 901, 40), ("bf16", 32, 8, 128, 9, 900, 640), ("bf16", 16, 8, 256, 7, 400, 40), ("bf16", 16, 8, 256, 11, 300, 40),
    ("f32", 16, 8, 128, 8, 300, 40), ("f32", 16, 8, 128, 12, 300, 700), ("bf16", 16, 4, 64, 7, 1100, 40), ("bf16", 16, 4, 64, 9, 1100, 40), ("bf16", 16, 4, 64, 17, 700, 600)])
def test_split_batches(dtype, hq, hkv, d, n, ctx, own):
    """Both sides of the lines between a CU's LDS for a workgroup, half of it, and the other kernels."""
    specs = [_spec(dtype, hq, hkv, d, (ctx - 3 * b - 40, 40 + 2 * b), 1, 11, own) for b in range(n)]
    rs = [W.make_request(s, DEV, request=b) for b, s in enumerate(specs)]
    lens = [own - (7 * b) % 40 for b in range(n)]
    out, lse = H.run_decode(specs[0], rs, lens)
    for b in range(n):
        _check(specs[b], rs[b], 1, lens[b], out[b], lse[b])


@pytest.mark.parametrize("dtype, hq, hkv, d, rows, lens", [
    ("bf16", 8, 2, 128, 8, (300, 460)), ("bf16", 8, 2, 128, 8, (213, 300)), ("bf16", 14, 2, 256, 5, (60, 150)), ("bf16", 8, 2, 64, 8, (1000, 24)), ("f32", 6, 2, 128, 12, (200, 32)),
    ("f32", 6, 1, 40, 9, (199, 1, 56))])
def test_few_tiles_split(dtype, hq, hkv, d, rows, lens):
    """Several tiles of 16 rows on an idle chip, one request and two, over the lengths at which more tiles run whole."""
    test_tiles_of_rows(dtype, hq, hkv, d, rows, lens)


@pytest.mark.parametrize("dtype, hq, hkv, d", [("bf16", 8, 2, 128), ("bf16", 4, 2, 256), ("bf16", 6, 2, 40), ("f32", 4, 2, 64), ("f32", 8, 2, 128)])
def test_tree_behind_long_own_streams(dtype, hq, hkv, d):
    lens = [50, 1, 128, 33, 300, 64, 2, 95]
    tree = W.tree_per_context(len(lens), 0.85)
    spec = _spec(dtype, hq, hkv, d, lens, 2, 20, 700)
    r = W.make_request(spec, DEV)
    h = H.HostArrays(r)
    for q_len in (1, 2):
        out, lse = H.run_tree(spec, r, tree, q_len, 702)
        ref, ref_lse = H.oracle_tree(h, q_len, 702, r.temperature, tree)
        H.check_close(H.f64(out).reshape(-1, d), ref, dtype, "tree")
        assert np.abs(H.f64(lse).T.reshape(-1) - ref_lse).max() <= H.lse_tol(dtype)
