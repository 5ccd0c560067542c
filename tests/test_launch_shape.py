"""Which kernel a decode call takes (host code, no GPU): the build with two sets of columns a workgroup serves neither a fp16 tail nor
three local tensors nor pairs of 64-channel heads, whatever the sizes."""
import ctypes as C
import random


def shape(dq, bits, group, rep, batch, tiles, heads=8, i3=1, tail=0, dim=128, flags=0):
    """(matrix-core kernel, splits, waves, query heads per workgroup)"""
    f, out = dq.Format(bits, group, dim, dim // 8, 8, 128, i3).c(), (C.c_int32 * 4)()
    assert dq.lib.dq_debug_decode_shape(C.byref(f), batch, heads * rep, heads, tiles * 128, tail, flags, out) == 0
    return tuple(out)


def test_two_sets_of_columns_take_no_tail_no_third_tensor_and_no_pairs(dq):
    rng = random.Random(1)
    wide = 0
    for _ in range(4000):
        bits, group, rep = rng.choice([2, 4, 8]), rng.choice([64, 128]), rng.randint(1, 16)
        batch, heads, tiles = rng.choice([1, 2, 5, 16, 64, 200]), 2 * rng.randint(1, 20), rng.choice([0, 1, 3, 4, 8, 33, 256, 1000])
        most = 4 if group == 128 else 2
        for tail, i3, dim in ((0, 1, 128), (1, 1, 128), (0, 8, 128), (1, 8, 128), (0, 1, 64), (1, 1, 64)):
            if dim == 64 and group != 64:
                continue
            mfma, splits, waves, per = shape(dq, bits, group, rep, batch, tiles, heads, i3, tail, dim)
            assert mfma and 1 <= splits <= max(tiles, 1) and waves in ((4,) if bits == 8 else (4, 8))
            assert per <= (2 if dim == 64 else most) or (per == 2 * most and not tail and i3 == 1 and dim == 128)
            if per > most:
                wide += 1
                assert -(-rep // most) % 2 == 0
    assert wide > 100


def test_the_plain_kernel_keeps_its_own_shape(dq):
    mfma, splits, waves, per = shape(dq, 4, 128, 8, 64, 64, flags=dq.DECODE_FORCE_GENERIC)
    assert not mfma and per == 8
