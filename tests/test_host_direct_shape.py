"""CPU: the workgroup shape of a prefill launch whose tiles go to LDS directly, against the general rule's; the block numbers that
a wave of it holds."""
import ctypes
import random

import numpy as np
import pytest

from test_host_rules import launch, lib, shape  # noqa: F401  (lib: a fixture)


def direct(lib, B, Hq, Hkv, max_q_len, whole=False, D=128, slopes=True, windowed=False, cus=256, key_bytes=0):
    return ["4", "8", "two"][lib.prefill_shape_direct_of(*launch(B, Hq, Hkv), max_q_len, D, slopes, windowed, whole, cus, ctypes.c_int64(key_bytes))]


@pytest.mark.parametrize("B,Hq,Hkv,max_q_len,whole,want", [
    (1, 32, 8, 1024, False, "two"), (1, 32, 8, 1025, False, "4"),
    (57, 32, 8, 64, False, "4"), (64, 32, 8, 64, False, "8"), (29, 32, 8, 65, False, "8"),       # 456 and 512 of one to a unit, 464 of two
    (6, 32, 8, 512, False, "4"), (7, 32, 8, 512, False, "8"), (8, 32, 8, 384, False, "4"), (8, 32, 8, 385, False, "8"),   # 384, 448
    (8, 32, 8, 3072, True, "4"), (8, 32, 8, 3073, True, "8"),
    (1, 32, 8, 8192, True, "4"), (2, 32, 8, 5120, True, "4"), (2, 32, 8, 5121, True, "8")])                              # 1 280, 1 296
def test_direct_shape(lib, B, Hq, Hkv, max_q_len, whole, want):
    assert direct(lib, B, Hq, Hkv, max_q_len, whole) == want
    for D, slopes in ((64, True), (64, False), (128, False)):
        assert direct(lib, B, Hq, Hkv, max_q_len, whole, D, slopes) == ("two" if want == "two" else "4")
    assert direct(lib, B, Hq, Hkv, max_q_len, whole, windowed=True) == "4"


FAR = 320000000                     # bytes of keys that the last-level cache does not keep


# (128-row workgroups no more than 256-row ones: one of 256 rows is half empty)
@pytest.mark.parametrize("B,Hq,Hkv,max_q_len,whole,key_bytes,want", [
    (64, 16, 16, 130, False, FAR - 1, "4"), (64, 16, 16, 130, False, FAR, "8"), (64, 16, 16, 128, False, FAR, "4"), (31, 16, 16, 256, False, FAR, "4"),
    (8, 32, 8, 2048, False, 0, "4"), (8, 32, 8, 2049, False, 0, "8"), (8, 32, 8, 2560, True, 0, "4"), (8, 32, 8, 8192, True, FAR - 1, "4"),
    (64, 16, 16, 1523, True, FAR, "8"), (40, 16, 16, 512, True, FAR, "4"), (40, 16, 16, 513, True, FAR, "8")])                 # 1 280 and 1 920
def test_direct_shape_without_slopes(lib, B, Hq, Hkv, max_q_len, whole, key_bytes, want):
    assert direct(lib, B, Hq, Hkv, max_q_len, whole, slopes=False, key_bytes=key_bytes) == want
    assert direct(lib, B, Hq, Hkv, max_q_len, whole, D=64, slopes=False, key_bytes=key_bytes) == "4"


def test_two_groups_and_windows_are_the_general_rules(lib):
    rng = random.Random(3)
    for _ in range(3000):
        Hkv = rng.choice([1, 2, 3, 8])
        args = rng.randint(1, 70), Hkv * rng.choice([1, 2, 3, 4, 7, 16, 17, 32]), Hkv, int(2 ** rng.uniform(0, 13))
        cus, windowed = rng.choice([64, 256, 304]), rng.random() < 0.3
        got = direct(lib, *args, rng.random() < 0.5, D=rng.choice([64, 128]), slopes=rng.random() < 0.5, windowed=windowed, cus=cus,
                     key_bytes=int(2 ** rng.uniform(20, 33)))
        any_ = shape(lib, *args, windowed=windowed, cus=cus)
        assert (got == "two") == (any_ == "two") and (not windowed or got == any_)


@pytest.mark.parametrize("back", [0, 1, 2, 5, 100])             # blocks that a walk started anew may go back by
def test_held_block_numbers(lib, back):
    """Down the blocks by 1 to 4 at a time, now and then on by many, or back by a few: the right number each time."""
    rng = random.Random(back)
    for _ in range(300):
        at = rng.randint(0, 3000)
        walk, step = [at], rng.randint(1, 4)
        while at > 0:
            at -= rng.randint(5, 300) if rng.random() < 0.02 else step
            if back and rng.random() < 0.05:
                at = min(at + rng.randint(1, back), walk[0])
            at = max(at, 0)
            walk.append(at)
        blocks, reads = np.array(walk, np.int32), ctypes.c_int()
        assert lib.held_blocks_differ(ctypes.c_void_p(blocks.ctypes.data), len(blocks), ctypes.byref(reads)) == -1
        assert back or reads.value <= 1 + walk[0] // 64
