"""CPU: the workgroup shape of a prefill launch whose tiles go to LDS directly, against the general rule's; the block numbers that
a wave of it holds."""
import ctypes
import random

import numpy as np
import pytest

from test_host_rules import lib, shape  # noqa: F401  (lib: a fixture)


def direct(lib, B, Hq, Hkv, max_q_len, whole=False, D=128, slopes=True, windowed=False, cus=256):
    group = Hq // Hkv
    gh = max(h for h in range(1, 17) if group % h == 0)
    units8 = -(-B * Hkv * (group // gh) // 8) * 8
    return ["4", "8", "two"][lib.prefill_shape_direct_of(ctypes.c_int64(units8), (gh - 1).bit_length(), max_q_len, D, slopes, windowed, whole, cus)]


@pytest.mark.parametrize("B,Hq,Hkv,max_q_len,whole,want", [
    (1, 32, 8, 1024, False, "two"), (1, 32, 8, 1025, False, "4"),
    (6, 32, 8, 512, False, "4"), (7, 32, 8, 512, False, "8"), (8, 32, 8, 384, False, "4"), (8, 32, 8, 385, False, "8"),   # 384, 448
    (8, 32, 8, 3072, True, "4"), (8, 32, 8, 3073, True, "8"),
    (1, 32, 8, 8192, True, "4"), (2, 32, 8, 5120, True, "4"), (2, 32, 8, 5121, True, "8")])                              # 1 280, 1 296
def test_direct_shape(lib, B, Hq, Hkv, max_q_len, whole, want):
    assert direct(lib, B, Hq, Hkv, max_q_len, whole) == want
    for D, slopes in ((64, True), (64, False), (128, False)):
        assert direct(lib, B, Hq, Hkv, max_q_len, whole, D, slopes) == ("two" if want == "two" else "4")
    assert direct(lib, B, Hq, Hkv, max_q_len, whole, windowed=True) == "4"


def test_two_groups_and_windows_are_the_general_rules(lib):
    rng = random.Random(3)
    for _ in range(3000):
        Hkv = rng.choice([1, 2, 3, 8])
        args = rng.randint(1, 70), Hkv * rng.choice([1, 2, 3, 4, 7, 16, 17, 32]), Hkv, int(2 ** rng.uniform(0, 13)), rng.random() < 0.5
        cus, windowed = rng.choice([64, 256, 304]), rng.random() < 0.3
        got = direct(lib, *args, D=rng.choice([64, 128]), slopes=rng.random() < 0.5, windowed=windowed, cus=cus)
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
