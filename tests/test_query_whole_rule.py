"""Host logic: which queries over short contexts run without splits.  The flash kernels' shapes leave their own kernels for that,
which has to pay for the rows and for the prefixes and own tokens as well.  The rule by itself: what the few-row kernels serve does not come to it (test_launch_layout.py)."""
import ctypes

import pytest

from paper_2502_05431_amd import binding as B


class ShapeInfo(ctypes.Structure):                        # csrc/ape_internal.h
    _fields_ = [(n, ctypes.c_int) for n in ("hq", "hkv", "d", "dtype", "group")] + [(n, ctypes.c_bool) for n in ("force_generic", "mfma", "tile")]


def _whole(batch, q_len, own, ctx=200, hq=32, hkv=8, d=128):
    lib = B.load()
    si = ShapeInfo()
    assert lib._ZN3ape11check_shapeEPK9ape_shapePNS_9ShapeInfoE(ctypes.byref(B.make_shape(hq, hkv, d, B.torch.bfloat16)), ctypes.byref(si)) == 0
    rule = lib._ZN3ape16whole_block_rowsERKNS_9ShapeInfoEiiill
    rule.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_long]
    return rule(ctypes.addressof(si), 1, batch, q_len, ctx, batch * own) > 0


@pytest.mark.parametrize("batch, q_len, own, whole", [
    (1, 1, 16000, True), (4, 1, 12000, True), (8, 1, 4000, True), (16, 1, 1500, True), (64, 1, 700, True),
    (8, 1, 12000, False), (16, 1, 4000, False), (32, 1, 4000, False), (64, 1, 1500, False),
    (1, 64, 1000, True), (1, 256, 16000, True), (3, 64, 4000, True), (16, 16, 1500, True),
    (16, 16, 4000, False), (8, 64, 64, False), (2, 256, 256, False), (1, 500, 500, False),
])
def test_flash_shapes(batch, q_len, own, whole):
    assert _whole(batch, q_len, own) == whole


@pytest.mark.parametrize("batch, q_len, whole", [(2, 64, True), (8, 64, False), (2, 256, False), (1, 100, True), (32, 1, True)])
def test_a_kv_head_has_one_xcd(batch, q_len, whole):
    assert _whole(batch, q_len, q_len, hq=16, hkv=2) == whole


@pytest.mark.parametrize("batch, q_len, own", [(32, 1, 4000), (4, 64, 64), (1, 250, 250)])
def test_other_shapes_have_no_other_kernel(batch, q_len, own):
    assert _whole(batch, q_len, own, ctx=100, hq=16, hkv=8, d=256)


@pytest.mark.parametrize("batch, q_len, ctx, own, whole", [
    (1, 1, 128, 160, True), (1, 1, 129, 129, False), (3, 1, 256, 400, False), (1, 16, 160, 200, False), (1, 1, 256, 128, True), (1, 1, 256, 1000, True),
    (12, 1, 256, 400, True), (1, 64, 200, 200, True),
])
def test_two_stages_on_both_sides(batch, q_len, ctx, own, whole):
    assert _whole(batch, q_len, own, ctx=ctx) == whole
