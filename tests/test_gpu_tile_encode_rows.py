"""GPU parity of the tile kernels' encode on every row tile and wavefront split it chooses between (32, 64 and 128 rows; tokens
or dims shared between wavefronts), at totals on both sides of the choices."""
import pytest

from paper_2502_05431_amd import workloads as W

import helpers as H
from test_gpu_parity import _check_encode

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype, hq, hkv, d", [("f32", 4, 2, 64), ("f32", 6, 2, 40), ("f32", 4, 2, 128), ("f32", 2, 2, 256),
                                               ("bf16", 4, 2, 64), ("bf16", 6, 2, 96), ("bf16", 4, 2, 256)])
@pytest.mark.parametrize("lens, prefix", [((1, 0, 31, 33), 0), ((200, 65, 130), 9), ((600, 1), 33), ((70,) * 45, 5), ((160,) * 70, 32)])
def test_row_tiles(dtype, hq, hkv, d, lens, prefix):
    spec = W.WorkloadSpec(name="rows", cfg=6, dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=prefix,
                          chunk_lens=tuple(lens), q_len=1, decode_steps=0)
    r = W.make_request(spec, DEV)
    _check_encode(spec, r, H.HostArrays(r), what="%s, %d lens" % (spec, len(lens)))
