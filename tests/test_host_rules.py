"""The rules that the host launches by and the index arithmetic that it prepares, run on the CPU: the library's own headers,
compiled for the host (tests/host_hip)."""
import ctypes
import os
import random
import subprocess
import types

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_02351_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "librules.so")
    clang = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    subprocess.run([clang, "-std=c++17", "-O1", "-fPIC", "-shared", "-Wno-ignored-attributes", "-I" + os.path.join(HERE, "host_hip"),
                    "-I" + CSRC, os.path.join(HERE, "host_hip", "rules.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def shape(lib, B, Hq, Hkv, max_q_len, whole_prompts=False, windowed=False, cus=256):
    group = Hq // Hkv
    gh = max(h for h in range(1, 17) if group % h == 0)
    units8 = -(-B * Hkv * (group // gh) // 8) * 8
    return ["4", "8", "two"][lib.prefill_shape_of(ctypes.c_int64(units8), (gh - 1).bit_length(), max_q_len, windowed, whole_prompts, cus)]


@pytest.mark.parametrize("B,Hq,Hkv,max_q_len,whole,want", [
    (1, 32, 8, 1024, False, "two"), (1, 32, 8, 1025, False, "4"),           # 256 and 264 workgroups of 128 rows
    (8, 32, 8, 448, False, "4"), (8, 32, 8, 449, False, "8"),               # 448 and 512 of 256 rows
    (8, 32, 8, 1280, True, "4"), (8, 32, 8, 1281, True, "8"),               # 1 280 and 1 344
    # a bound of 2 048 and more may stand over prompts of any length: no line there
    (4, 32, 8, 2047, True, "4"), (4, 32, 8, 2048, True, "4"), (4, 32, 8, 2560, True, "4"), (2, 32, 8, 4096, True, "4"),
    (1, 32, 8, 8192, True, "4"), (4, 32, 4, 2560, True, "4"), (8, 32, 8, 2560, True, "8")])
def test_prefill_shape(lib, B, Hq, Hkv, max_q_len, whole, want):
    assert shape(lib, B, Hq, Hkv, max_q_len, whole) == want
    assert shape(lib, B, Hq, Hkv, max_q_len, windowed=True) == "4"


def test_the_gpu_tests_know_the_rule(lib, monkeypatch):
    """launch_shape, by which the GPU tests choose their launches, against the rule itself."""
    import torch
    from test_gpu_prefill_walk import launch_shape
    rng = random.Random(1)
    seen = set()
    for _ in range(3000):
        cus = rng.choice([64, 256, 304])
        monkeypatch.setattr(torch.cuda, "get_device_properties", lambda _: types.SimpleNamespace(multi_processor_count=cus))
        Hkv = rng.choice([1, 2, 3, 8])
        args = rng.randint(1, 70), Hkv * rng.choice([1, 2, 3, 4, 7, 16, 17, 32]), Hkv, int(2 ** rng.uniform(0, 13)), rng.random() < 0.5
        got = launch_shape(*args)[0]
        assert got == shape(lib, *args, cus=cus), (args, cus)
        seen.add(got)
    assert seen == {"two", "4", "8"}
