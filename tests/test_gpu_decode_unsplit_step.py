"""GPU parity of the one-call decode step where the context is not split: the kernel that attends stores the
new rows itself (one workgroup per KV head, few sequences), or a launch in front of it does."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U, oracle_filled  # noqa: F401  (U: a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv,D", [
    (W.F16, 8, 2, 64), (W.BF16, 16, 2, 64),                  # group 4 and 8: ring kernel
    (W.F16, 6, 3, 64), (W.BF16, 3, 3, 64),                   # group 2 and 1: general kernel
    (W.F16, 6, 2, 64), (W.BF16, 32, 2, 64),                  # group 3 and 16: several workgroups a group, own launch
    (W.BF16, 8, 2, 128), (W.F16, 3, 1, 128), (W.BF16, 16, 1, 128), (W.F16, 20, 1, 128),   # 20: two workgroups
])
def test_unsplit_step(U, oracle, dtype, Hq, Hkv, D):
    """Lengths at block and tile edges, 1 and 0; new rows dense and as strided views; caches bit for bit
    (the new rows hold NaN patterns until the step stores them)."""
    import torch
    import paper_2505_02351_amd as G
    lens = np.array([128, 1, 16, 17, 0, 31, 33, 127, 256], np.int32)
    B = len(lens)
    cfg = W.small_config(name="unsplit", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=16,
                         num_blocks=B * 17, ctx_lo=1, ctx_hi=256, seed=Hq + D)
    case = W.make_case(cfg, context_lens=lens)
    kc, vc = oracle_filled(oracle, case)

    def full(a):
        z = np.zeros((B,) + a.shape[1:], np.uint16)
        z[lens > 0] = a
        return z
    k_new, v_new = full(case.k_new), full(case.v_new)
    case.q = full(case.q)
    ref = oracle.paged_attention(case.q, kc, vc, case.block_tables, case.context_lens, case.slopes, case.scale, dtype)
    assert G.paged_attention_workspace_bytes(B, Hq, Hkv, D, 16, 256, 0) == (0, 0)
    for pad in (0, 8, 1):                                    # token strides: dense, a multiple of 8 elements, odd
        dev = U.DevCase(case)
        rows = []
        for a in (k_new, v_new):
            wide = torch.zeros(B, Hkv * D + pad, dtype=dev.q.dtype, device="cuda")
            wide[:, :Hkv * D] = U.to_dev(a, dtype).reshape(B, Hkv * D)
            rows.append(wide[:, :Hkv * D].unflatten(1, (Hkv, D)))
        dev.k_new, dev.v_new = rows
        assert U.max_abs_err(dev.step(None), ref, dtype) <= U.TOL[dtype], pad
        assert np.array_equal(U.to_host(dev.k_cache), kc) and np.array_equal(U.to_host(dev.v_cache), vc), pad


@pytest.mark.parametrize("n", [2, 32, 33, 40])                 # 32 sequences: the most that one launch serves
@pytest.mark.parametrize("dtype,Hq,Hkv,D", [(W.F16, 8, 2, 64), (W.BF16, 4, 2, 64), (W.BF16, 8, 2, 128)])
def test_tokens_of_one_sequence_as_batch_entries(U, oracle, dtype, Hq, Hkv, D, n):
    """The step's n new tokens are successive tokens of ONE sequence (same block table, lengths one apart): every
    entry sees the new rows of those before it, as if all rows had been written first."""
    lens = np.arange(61, 61 + n, dtype=np.int32)
    cfg = W.small_config(name="successive", dtype=dtype, batch=n, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=16,
                         num_blocks=n * 8, ctx_lo=1, ctx_hi=128, seed=n + D)
    case = W.make_case(cfg, context_lens=lens)
    case.block_tables[:] = case.block_tables[-1]
    pos = lens - 1
    blk, row = case.block_tables[0, pos // 16], pos % 16
    case.k_cache[blk, :, row] = case.v_cache[blk, :, row] = W.NAN_BITS[dtype]
    case.slot_mapping = blk.astype(np.int64) * 16 + row
    kc, vc = oracle_filled(oracle, case)
    ref = oracle.paged_attention(case.q, kc, vc, case.block_tables, case.context_lens, case.slopes, case.scale, dtype)
    dev = U.DevCase(case)
    assert U.max_abs_err(dev.step(None), ref, dtype) <= U.TOL[dtype]
    assert np.array_equal(U.to_host(dev.k_cache), kc) and np.array_equal(U.to_host(dev.v_cache), vc)


def microseconds(call, reps=20, runs=7):
    """GPU time of one of `reps` back-to-back calls, the best of several runs."""
    import torch
    call()
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = float("inf")
    for _ in range(runs):
        torch.cuda.synchronize()
        a.record()
        for _ in range(reps):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / reps)
    return best


@pytest.mark.parametrize("Hq,Hkv,D,limit", [(16, 4, 128, 0.95), (8, 8, 64, 1.25)])
def test_unsplit_attention_keeps_its_tiles_in_flight(U, Hq, Hkv, D, limit):
    """64 sequences of 1 000 tokens without a split, against the equal-work split of the same call: 0.82 and
    1.04 of its time; 1.08 and 1.50 when a block number is a vector load that waits for the tiles in flight."""
    import paper_2505_02351_amd as G
    cfg = W.small_config(name="in flight", dtype=W.F16, batch=64, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=16,
                         num_blocks=64 * 63 + 8, ctx_lo=1000, ctx_hi=1000, seed=5)
    dev = U.DevCase(W.make_case(cfg))
    dev.write_cache()
    ws = dev.workspace(G.SPLIT_BALANCED)[0]
    unsplit, split = (microseconds(lambda: G.paged_attention(dev.out, dev.q, dev.k_cache, dev.v_cache, dev.block_tables,
                                                             dev.context_lens, dev.slopes, float(dev.case.scale), 1000, how, ws))
                      for how in (-1, G.SPLIT_BALANCED))
    assert unsplit <= limit * split, (unsplit, split)
