"""The rules that the host launches by and the index arithmetic that it prepares, run on the CPU: the library's own headers,
compiled for the host (tests/host_hip)."""
import ctypes
import os
import random
import subprocess
import types

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_02351_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "librules.so")
    clang = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    # (-O0: a load whose value is not used must stay)
    subprocess.run([clang, "-std=c++17", "-O0", "-fPIC", "-shared", "-Wno-ignored-attributes", "-I" + os.path.join(HERE, "host_hip"),
                    "-I" + CSRC, "-I" + os.path.join(os.path.dirname(HERE), "include"), os.path.join(HERE, "host_hip", "rules.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def ptr(a):
    return None if a is None else ctypes.c_void_p(a.ctypes.data)


def test_division_by_the_hosts_reciprocal(lib):
    """All of 0 <= n < 2^31: ends and neighbours of multiples, for divisors that occur and for the largest."""
    f = lib.fast_div_differs
    f.restype = ctypes.c_int64
    rng = np.random.default_rng(1)
    divisors = {1, 2, 3, 2**31 - 1, 2**31 - 2} | {(1 << s) + d for s in range(2, 31) for d in (-1, 0, 1)}
    divisors = sorted(divisors | set(range(1, 300)) | {int(x) for x in np.exp2(rng.uniform(0, 31, 2000))})
    top = 2**31 - 1
    for d in divisors:
        q = np.unique(np.concatenate([[0, 1, top // d], rng.integers(0, top // d + 1, 40)]))
        n = np.concatenate([q * d - 1, q * d, q * d + d - 1, [top, top - 1], rng.integers(0, top, 20)])
        n = np.ascontiguousarray(n[(n >= 0) & (n <= top)], np.int32)
        at = f(ptr(np.array([d], np.uint32)), 1, ptr(n), len(n))
        assert at < 0, (d, n[at])


@pytest.mark.parametrize("ulps", [-2, -1, 0, 1, 2])         # v_rcp_f32 is good to one; the product rounds once more
def test_division_by_a_rounded_inverse(lib, ulps):
    """Quotients below 2^20 (those of the combine kernel are waves of a launch, a few thousand), numerators up to 2^30."""
    f = lib.div_by_inverse_differs
    f.restype = ctypes.c_int64
    rng = np.random.default_rng(2)
    for d in sorted(set(range(1, 200)) | {int(x) for x in np.exp2(rng.uniform(0, 30, 2000))}):
        top = min(2**30 // d, 2**20 - 1)
        q = np.unique(np.concatenate([[0, 1, top], rng.integers(0, top + 1, 40)]))
        n = np.concatenate([q * d - 1, q * d, q * d + d - 1])
        n = np.ascontiguousarray(n[n >= 0], np.int32)
        at = f(ptr(np.array([d], np.int32)), 1, ptr(n), len(n), ulps)
        assert at < 0, (d, n[at])


# (kinds: 16-byte pieces, single elements, E4M3 codes - whose decode step stores its rows in the combine kernel)
@pytest.mark.parametrize("kind,decode", [(0, False), (0, True), (1, False), (1, True), (2, False)])
@pytest.mark.parametrize("Hkv,D,bs", [(1, 64, 16), (3, 128, 32), (5, 64, 64)])
@pytest.mark.parametrize("slice_tokens", [1, 3, 8, None])       # tokens to a launch
def test_cache_stores_slice_by_slice(lib, slice_tokens, decode, kind, Hkv, D, bs):
    """Rows land where their slots say however the launches are cut; the rows of padding tokens (of empty sequences, in a
    decode step) beyond those that there are, which a graph's fixed batch has, are not read."""
    rng = np.random.default_rng(7 * Hkv + bs + kind)
    tokens, rows, pool = 17, 13, 9
    pad = 1 if kind == 1 else 8
    ks, vs = Hkv * D + pad, Hkv * D + 2 * pad
    k, v = (rng.integers(0, 100, (rows, s)).astype(np.float32) for s in (ks, vs))
    k, v = ((x.view(np.uint32) >> 16).astype(np.uint16) for x in (k, v))    # bf16
    dt = np.uint8 if kind == 2 else np.uint16
    got = [np.full((pool + 2, Hkv, bs, D), 255, dt) for _ in range(2)]      # a block ahead of the cache and one behind it
    want = [x.copy() for x in got]
    slots = np.full(tokens, -1, np.int64)
    slots[:rows] = rng.permutation(pool * bs)[:rows]
    slots[2] = -1                                               # and one among them
    tables, lens = np.full((tokens, 4), -1, np.int32), np.zeros(tokens, np.int32)
    for t in range(tokens):
        if slots[t] >= 0:
            block = int(rng.integers(4))
            tables[t, block], lens[t] = slots[t] // bs, block * bs + slots[t] % bs + 1
    tables[4, (lens[4] - 1) // bs] = -1                         # no block: nothing is stored (decode)
    for c, x in zip(want, (k, v)):
        for t in range(rows):
            if slots[t] >= 0 and not (decode and t == 4):
                row = x[t, :Hkv * D].reshape(Hkv, D)
                c[1 + slots[t] // bs, :, slots[t] % bs] = (row.astype(np.uint32) << 16).view(np.float32).astype(dt) if kind == 2 else row
    per_token = Hkv * D // (1 if kind == 1 else 8)
    most = 2**31 - 1 if slice_tokens is None else per_token * slice_tokens + per_token - 1
    n = lib.cache_store(kind, ptr(k), ptr(v), rows, ctypes.c_int64(ks), ctypes.c_int64(vs), ptr(got[0][1:]), ptr(got[1][1:]),
                        None if decode else ptr(slots), ptr(tables), ptr(lens), 4, tokens, Hkv, D, bs, most)
    assert n == (1 if slice_tokens is None else -(-tokens // slice_tokens))
    assert (got[0] == want[0]).all() and (got[1] == want[1]).all()


def test_cache_slices_and_refusals(lib):
    first, pieces = np.zeros(300, np.int64), np.zeros(300, np.int64)

    def slices(tokens, Hkv, D, elems):
        n = lib.cache_slices(ctypes.c_int64(Hkv * D), tokens, Hkv, D, elems, ptr(first), ptr(pieces), 300)
        return n if n < 0 else [(int(a), int(b)) for a, b in zip(first[:n], pieces[:n])]
    assert slices(4096, 8, 128, 8) == [(0, 4096 * 128)]
    assert slices(2**24 - 1, 8, 128, 8) == [(0, 2**31 - 128)]   # 128 pieces to a token: the most that one launch takes
    assert slices(2**24, 8, 128, 8) == [(0, 2**31 - 128), (2**24 - 1, 128)]
    assert slices(5, 2**24 - 1, 128, 1) == [(t, 2**31 - 128) for t in range(5)]
    assert slices(1, 2**24, 128, 1) == -2                       # one token is too much for a launch
    most = (2**31 - 1) * 128 // 1024                            # tokens of 1024 pieces
    assert len(slices(most, 8, 128, 1)) == 129 and slices(most + 1, 8, 128, 1) == -2


@pytest.mark.parametrize("Hkv,D,bs", [(1, 64, 16), (3, 128, 32), (5, 64, 64), (2, 128, 16)])
@pytest.mark.parametrize("seqs", [1, 4, 17, 32])
def test_a_steps_store_of_its_new_rows(lib, seqs, Hkv, D, bs):
    """store_new_rows: every sequence's row in its block; the rows of empty sequences, which need not exist, are not read."""
    rng = np.random.default_rng(seqs + Hkv)
    ks, vs, pool = Hkv * D + 8, Hkv * D, seqs + 3
    lens = rng.integers(0, 4 * bs, seqs).astype(np.int32)
    rows = max(seqs - 3, 1)
    lens[rows:] = 0                                             # the last ones are a graph's padding
    tables = np.full((seqs, 4), -1, np.int32)
    tables[np.arange(seqs), np.maximum(lens - 1, 0) // bs] = rng.permutation(pool)[:seqs]
    k, v = (rng.integers(0, 2**16, (rows, s)).astype(np.uint16) for s in (ks, vs))
    got = [np.zeros((pool, Hkv, bs, D), np.uint16) for _ in range(2)]
    want = [x.copy() for x in got]
    for b in np.flatnonzero(lens > 0):
        pos = lens[b] - 1
        for c, x in zip(want, (k, v)):
            c[tables[b, pos // bs], :, pos % bs] = x[b, :Hkv * D].reshape(Hkv, D)
    assert lib.step_store(ptr(k), ptr(v), rows, ctypes.c_int64(ks), ctypes.c_int64(vs), ptr(got[0]), ptr(got[1]), ptr(tables), ptr(lens), 4,
                          seqs, Hkv, D, bs) == 1
    assert (got[0] == want[0]).all() and (got[1] == want[1]).all()


def launch(B, Hq, Hkv):
    """A launch's (units8, heads_pow2_shift)."""
    group = Hq // Hkv
    gh = max(h for h in range(1, 17) if group % h == 0)
    return ctypes.c_int64(-(-B * Hkv * (group // gh) // 8) * 8), (gh - 1).bit_length()


def shape(lib, B, Hq, Hkv, max_q_len, windowed=False, cus=256):
    return ["4", "8", "two"][lib.prefill_shape_of(*launch(B, Hq, Hkv), max_q_len, windowed, cus)]


@pytest.mark.parametrize("B,Hq,Hkv,max_q_len,want", [
    (1, 32, 8, 1024, "two"), (1, 32, 8, 1025, "4"),                         # 256 and 264 workgroups of 128 rows
    (8, 32, 8, 448, "4"), (8, 32, 8, 449, "8"), (8, 32, 8, 2560, "8")])     # 448 and 512 of 256 rows
def test_prefill_shape(lib, B, Hq, Hkv, max_q_len, want):
    assert shape(lib, B, Hq, Hkv, max_q_len) == want
    assert shape(lib, B, Hq, Hkv, max_q_len, windowed=True) == "4"


def test_the_gpu_tests_know_the_rule(lib, monkeypatch):
    """launch_shape and launch_deep, by which the GPU tests choose their launches, against the rules themselves."""
    import torch
    from test_gpu_prefill_walk import launch_deep, launch_shape
    rng = random.Random(1)
    seen, deep = {}, {}
    for _ in range(6000):
        cus = rng.choice([64, 256, 304])
        monkeypatch.setattr(torch.cuda, "get_device_properties", lambda _: types.SimpleNamespace(multi_processor_count=cus))
        Hkv = rng.choice([1, 2, 3, 8])
        args = rng.randint(1, 70), Hkv * rng.choice([1, 2, 3, 4, 7, 16, 17, 32]), Hkv, int(2 ** rng.uniform(0, 13))
        kv8, D, slopes, longest = rng.random() < 0.3, rng.choice([64, 128]), rng.random() < 0.5, int(2 ** rng.uniform(5, 16))
        whole = not kv8 and rng.random() < 0.4
        window = 0 if kv8 or whole or rng.random() < 0.7 else int(2 ** rng.uniform(4, 13))
        keys = args[0] * (min(longest, window + args[3]) if window else longest)
        how = dict(D=D, slopes=slopes, kv8=kv8, window=window, longest=longest)
        got = launch_shape(*args, whole, **how)[0]
        if kv8:
            assert got == shape(lib, *args, cus=cus), (args, cus)
        else:
            want = lib.prefill_shape_direct_of(*launch(*args[:3]), args[3], D, slopes, window > 0, whole, cus, ctypes.c_int64(4 * Hkv * D * keys))
            assert got == ["4", "8", "two"][want], (args, whole, how, cus)
            if not whole:
                two_ahead = bool(lib.prefill_deep_of(*launch(*args[:3]), args[3], slopes, window > 0, cus, ctypes.c_int64(keys // args[0])))
                assert launch_deep(*args, **{k: v for k, v in how.items() if k not in ("kv8", "D")}) == two_ahead
                deep[got, two_ahead] = deep.get((got, two_ahead), 0) + 1
        seen[got, kv8, whole, slopes] = seen.get((got, kv8, whole, slopes), 0) + 1
    assert {s for s, *_ in seen} == {"two", "4", "8"} and len(deep) == 6
    assert {k[1:] for k in seen if k[0] == "8"} == {(True, False, True), (True, False, False), (False, False, True), (False, False, False),
                                                    (False, True, True), (False, True, False)}


def test_the_gpu_tests_know_when_units_are_taken_in_pairs(lib):
    from test_gpu_decode_pairs import pairs_from
    rng = random.Random(2)
    seen = [0, 0]
    for _ in range(3000):
        cus, Hkv = rng.choice([64, 256, 304]), rng.choice([1, 2, 3, 8])
        B, Hq, bound = rng.randint(1, 400), Hkv * rng.choice([1, 2, 4, 7, 16, 17, 32]), int(2 ** rng.uniform(4, 17))
        group = Hq // Hkv
        segments = B * Hkv * (group // max(h for h in range(1, 17) if group % h == 0))
        got = lib.decode_pairs_from_of(ctypes.c_int64(segments), ctypes.c_int64(B * Hq), bound, cus)
        assert got == pairs_from(B, Hq, Hkv, bound, cus)
        seen[got > 0] += 1
    assert min(seen) > 300
    assert lib.decode_pairs_from_of(ctypes.c_int64(2**26), ctypes.c_int64(2**30), 256, 256) == 2**31 - 1      # beyond any launch's tiles: never taken
