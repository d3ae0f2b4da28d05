"""GPU parity of the fp32 encode in three bf16 pieces (up to 128 dims): both row tiles it has, padded widths, streams that end inside a stage,
and the values that its pieces cannot carry: infinities, values that are none, the lowest of the type, and values below what bf16 holds."""
import numpy as np
import pytest
import torch

from paper_2502_05431_amd import workloads as W

import helpers as H
from test_gpu_parity import _check_encode

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _spec(hq, hkv, d, lens, prefix):
    return W.WorkloadSpec(name="split", cfg=6, dtype="f32", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=prefix, chunk_lens=tuple(lens),
                          q_len=1, decode_steps=0)


@pytest.mark.parametrize("hq, hkv, d, lens, prefix", [
    # 128 rows
    (8, 2, 128, (600, 1, 333) * 5, 7), (6, 6, 96, (129, 31, 0, 500) * 10, 33), (16, 2, 128, (90,) * 24, 0), (4, 4, 40, (300, 77) * 20, 31),
    (8, 2, 64, (33, 95, 160) * 14, 64), (3, 1, 8, (5000, 4001), 1),
    # 64 rows, two wavefronts a run of tokens apart
    (8, 2, 128, (1100, 900, 1), 5), (4, 4, 72, (1025, 1023, 601), 32), (4, 2, 64, (64, 31, 1, 100) * 16, 9), (6, 2, 40, (1000, 999, 1500), 0),
])
def test_tiles(hq, hkv, d, lens, prefix):
    spec = _spec(hq, hkv, d, lens, prefix)
    r = W.make_request(spec, DEV)
    _check_encode(spec, r, H.HostArrays(r), what=str(spec))


def _encode(r, spec, generic=False):
    o, lse, _, _ = H.run_encode(spec, r, generic=generic, with_prefix_rows=False)
    return H.f64(o), H.f64(lse)


@pytest.mark.parametrize("hq, hkv, d, lens", [(8, 2, 128, (700, 500) * 4), (8, 2, 64, (500, 400, 450) * 4), (4, 4, 128, (1000, 990), )])
@pytest.mark.parametrize("what", ["v_inf", "v_nan", "k_inf", "k_lowest", "v_lowest", "v_tiny", "v_zero"])
def test_values(hq, hkv, d, lens, what):
    """Against the vector-ALU kernels (plain fp32 products): the same rows are numbers, infinite or none, and the numbers agree."""
    spec = _spec(hq, hkv, d, lens, 9)
    r = W.make_request(spec, DEV)
    at = 300
    low = torch.finfo(torch.float32).min
    if what == "v_inf":
        r.v_ctx[at, 0, 3] = float("inf")
    elif what == "v_nan":
        r.v_ctx[at, 0, 3] = float("nan")
    elif what == "k_inf":
        r.k_ctx[at, 0, 5] = float("-inf")
    elif what == "k_lowest":                                # a score of -inf or +inf, as q goes
        r.k_ctx[at, 0, 5] = low
    elif what == "v_lowest":
        r.v_ctx[at, :, 2] = low
    elif what == "v_tiny":
        r.v_ctx.mul_(1e-35)
        r.v_prefix.mul_(1e-35)
    else:
        r.v_ctx.zero_()
        r.v_prefix.zero_()
    o, lse = _encode(r, spec)
    ref, ref_lse = _encode(r, spec, generic=True)
    assert np.array_equal(np.isnan(o), np.isnan(ref)) and np.array_equal(np.isinf(o), np.isinf(ref))
    ok = np.isfinite(ref)
    if what == "v_lowest":                                   # (of the magnitude of the type's range in that dim)
        o, ref = np.clip(o, -1e30, 1e30), np.clip(ref, -1e30, 1e30)
    scale = 1e-35 if what == "v_tiny" else 1.0
    # an fp32 path each: twice the bound of one against the oracle
    assert np.abs(o[ok] - ref[ok]).max() <= 2e-5 * scale
    ok = np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(lse), ok) and np.abs(lse[ok] - ref_lse[ok]).max() <= 2 * H.lse_tol("f32")
