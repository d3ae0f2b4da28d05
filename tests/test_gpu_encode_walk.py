"""GPU parity of the encode that walks several query tiles of a short context per workgroup, where it can go wrong: tiles
with one, two and many blocks (what is in flight at a tile's start differs), a prefix that ends inside a block, ragged and
empty contexts, lengths on both sides of the switches to the kernel of long contexts and between the numbers of tiles a
workgroup walks."""
import pytest

from paper_2502_05431_amd import workloads as W

import helpers as H
from test_gpu_parity import _check_encode

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(hq, hkv, lens, prefix):
    spec = W.WorkloadSpec(name="walk", cfg=6, dtype="bf16", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, prefix_len=prefix,
                          chunk_lens=tuple(lens), q_len=1, decode_steps=0)
    r = W.make_request(spec, DEV)
    _check_encode(spec, r, H.HostArrays(r), what="%d/%d heads, %s, prefix %d" % (hq, hkv, lens, prefix))


@pytest.mark.parametrize("hq, hkv", [(2, 2), (4, 2), (8, 2), (16, 2)])
@pytest.mark.parametrize("prefix", [0, 1, 31, 32, 33, 100])
def test_tile_and_block_edges(hq, hkv, prefix):
    _check(hq, hkv, (1, 16, 31, 32, 33, 0, 64, 65, 127, 129, 255, 257), prefix)


@pytest.mark.parametrize("n, chunk_len", [(3, 512), (3, 513), (200, 96), (60, 70), (40, 40), (9, 900), (600, 33)])
def test_work_splits(n, chunk_len):
    _check(8, 2, [max(0, chunk_len - 5 * (i % 7)) for i in range(n)], 7)


def test_many_ragged_contexts():
    _check(32, 8, [1 + (37 * i) % 300 for i in range(300)], 32)


@pytest.mark.parametrize("hq, hkv, lens, prefix", [(32, 8, (512,) * 8, 5), (8, 2, (96,) * 40, 300), (8, 2, (96,) * 40, 600), (8, 2, (200, 300), 1100)])
def test_prefixes_on_both_sides_of_the_switch(hq, hkv, lens, prefix):
    _check(hq, hkv, lens, prefix)
