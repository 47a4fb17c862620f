"""GPU parity of the combine that reads a head's partial results with eight groups of threads: few sequences,
contexts of many pieces (and of few, of one token, of none), every form of the decode that ends in it."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import BALANCED, U, oracle_filled  # noqa: F401  (U: a fixture)

pytestmark = pytest.mark.gpu

LENS = {1: [4101], 2: [6000, 1], 5: [3333, 0, 17, 900, 32]}


def make(B, dtype, Hq, Hkv, D, seed):
    lens = np.array(LENS[B], np.int32)
    cfg = W.small_config(name="pieces", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=16,
                         num_blocks=int((lens // 16 + 1).sum()) + 5, ctx_lo=1, ctx_hi=int(lens.max()), seed=seed)
    case = W.make_case(cfg, context_lens=lens)
    if case.q.shape[0] != B:                    # sequences without tokens have no rows: give them some
        def full(a):
            z = np.zeros((B,) + a.shape[1:], np.uint16)
            z[lens > 0] = a
            return z
        rows = (full(case.q), full(case.k_new), full(case.v_new))
    else:
        rows = (case.q, case.k_new, case.v_new)
    return case, rows


@pytest.mark.parametrize("B", [1, 2, 5])
@pytest.mark.parametrize("dtype,Hq,Hkv,D", [(W.BF16, 8, 2, 128), (W.F16, 6, 2, 64), (W.F16, 20, 1, 128)])
def test_many_pieces(U, oracle, dtype, Hq, Hkv, D, B):
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    import pins_e4m3
    case, (q, k_new, v_new) = make(B, dtype, Hq, Hkv, D, 31 * B + D)
    kc, vc = oracle_filled(oracle, case)
    ref = oracle.paged_attention(q, kc, vc, case.block_tables, case.context_lens, case.slopes, case.scale, dtype)
    case.q = q
    dev = U.DevCase(case)
    dev.k_new, dev.v_new = U.to_dev(k_new, dtype), U.to_dev(v_new, dtype)
    assert U.max_abs_err(dev.step(dev.workspace(BALANCED)[0]), ref, dtype) <= U.TOL[dtype]
    assert np.array_equal(U.to_host(dev.k_cache), kc) and np.array_equal(U.to_host(dev.v_cache), vc)
    for partition in (BALANCED, 16, 64, 512):
        assert U.max_abs_err(dev.decode(partition_size=partition), ref, dtype) <= U.TOL[dtype], partition
    ref_w = O.paged_attention_window(q, kc, vc, case.block_tables, case.context_lens, case.slopes, case.scale, 2500, dtype)
    assert U.max_abs_err(dev.decode_window(2500), ref_w, dtype) <= U.TOL[dtype]
    # 8-bit step: the new token's term is added behind the merge
    k_scale, v_scale = 0.0125, 0.0125
    kc8, vc8, _ = pins_e4m3.quantised_cache(case, k_scale, v_scale)
    k_old, v_old, slots_old = W.all_token_rows(case, include_new=False)
    dk = torch.full(kc8.shape, 0x7F, dtype=torch.uint8, device="cuda")
    dv = torch.full(vc8.shape, 0x7F, dtype=torch.uint8, device="cuda")
    G.reshape_and_cache_fp8(U.to_dev(k_old, dtype), U.to_dev(v_old, dtype), dk, dv, torch.from_numpy(slots_old).cuda(), k_scale, v_scale)
    dev.out.fill_(float("nan"))
    G.decode_step_fp8(dev.out, dev.q, dev.k_new, dev.v_new, dk, dv, dev.block_tables, dev.context_lens, dev.slopes,
                      float(case.scale), k_scale, v_scale, case.max_context_len, dev.workspace(BALANCED)[0])
    torch.cuda.synchronize()
    dev.check_canaries()
    assert np.array_equal(dk.cpu().numpy(), kc8) and np.array_equal(dv.cpu().numpy(), vc8)
    ref8 = O.paged_attention_e4m3(q, kc8, vc8, case.block_tables, case.context_lens, case.slopes, case.scale, k_scale, v_scale, dtype)
    assert U.max_abs_err(U.to_host(dev.out), ref8, dtype) <= U.TOL[dtype]


def test_many_pieces_behind_a_shared_prefix(U, oracle):
    """Four sequences of 3 000 and some tokens with 2 000 of them in common (bundles of 4)."""
    cfg = W.small_config(name="pieces_shared", dtype=W.BF16, batch=4, num_heads=16, num_kv_heads=4, head_dim=128, block_size=16,
                         num_blocks=4 * 210, ctx_lo=3001, ctx_hi=3200, seed=10)
    case = W.make_case(cfg)
    shared = np.array([0, 125, 125, 125], np.int32)
    case.block_tables[1:, :125] = case.block_tables[0, :125]
    kc, vc = oracle_filled(oracle, case)
    ref = oracle.paged_attention(case.q, kc, vc, case.block_tables, case.context_lens, case.slopes, case.scale, W.BF16)
    dev = U.DevCase(case)
    assert U.max_abs_err(dev.decode_shared(shared, fused=True), ref, W.BF16) <= U.TOL[W.BF16]
    assert U.max_abs_err(dev.decode_shared(shared), ref, W.BF16) <= U.TOL[W.BF16]


@pytest.mark.parametrize("B", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("Hq,Hkv,D", [(8, 2, 128), (6, 2, 64), (8, 8, 64)])      # bundles of 4, 5 and 16
def test_shared_prefixes_at_the_lane_limit(U, oracle, B, Hq, Hkv, D):
    """Up to 64 sequences keep their extents in lanes, more read them from memory: random shares,
    members that share nothing."""
    rng = np.random.default_rng(B + D)
    lens = rng.integers(1, 150, B).astype(np.int32)
    cfg = W.small_config(name="lanes", dtype=W.F16, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=16,
                         num_blocks=B * 11, ctx_lo=1, ctx_hi=150, seed=B)
    case = W.make_case(cfg, context_lens=lens)
    bundle = 16 // (Hq // Hkv)
    shared = np.zeros(B, np.int32)
    for b in range(B):
        b0 = b - b % bundle
        if b != b0 and rng.random() < 0.7:
            shared[b] = rng.integers(0, min(lens[b] - 1, lens[b0] - 1) // 16 + 1)
            case.block_tables[b, :shared[b]] = case.block_tables[b0, :shared[b]]
    kc, vc = oracle_filled(oracle, case)
    ref = oracle.paged_attention(case.q, kc, vc, case.block_tables, case.context_lens, case.slopes, case.scale, W.F16)
    dev = U.DevCase(case)
    assert U.max_abs_err(dev.decode_shared(shared, fused=True), ref, W.F16) <= U.TOL[W.F16]
    assert np.array_equal(U.to_host(dev.k_cache), kc) and np.array_equal(U.to_host(dev.v_cache), vc)
    assert U.max_abs_err(dev.decode_shared(shared), ref, W.F16) <= U.TOL[W.F16]
