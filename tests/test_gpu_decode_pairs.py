"""GPU parity of decode over 8-bit caches where a wave takes two tiles at a time (head_dim 128, long units under the caller's bound):
units of one, few and many tiles, odd ones among them, sequences of one token, several pieces to a unit."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu
BOUND = 4096                        # 16 sequences x 8 KV heads x 256 tiles: 32 tiles to each of 1 024 units


@pytest.mark.parametrize("lo,hi", [(1, 5), (1, 70), (15, 700), (1, 4096), (4081, 4096)])
@pytest.mark.parametrize("Hq,block_size", [(8, 16), (32, 64)])
@pytest.mark.parametrize("dtype", [W.BF16, W.F16])
def test_two_tiles_at_a_time(U, oracle, dtype, Hq, block_size, lo, hi):
    import torch
    import oracle as O
    import pins_e4m3
    import paper_2505_02351_amd as G
    B, Hkv, D, k_scale, v_scale = 16, 8, 128, 0.0125, 0.03
    assert B * Hkv * (BOUND // 16) >= 32 * 4 * torch.cuda.get_device_properties(0).multi_processor_count
    cfg = W.small_config(name="pairs", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=block_size,
                         num_blocks=B * -(-hi // block_size) + 7, ctx_lo=lo, ctx_hi=hi, seed=hi + Hq)
    case = W.make_case(cfg)
    kc8, vc8, (k_all, v_all, slots) = pins_e4m3.quantised_cache(case, k_scale, v_scale)
    case.block_tables = np.pad(case.block_tables, ((0, 0), (0, BOUND // block_size - case.block_tables.shape[1])), constant_values=-1)
    ref = O.paged_attention_e4m3(case.q, kc8, vc8, case.block_tables, case.context_lens, case.slopes, case.scale, k_scale, v_scale, dtype)
    dev = U.DevCase(case)
    ws = torch.empty(G.paged_attention_workspace_bytes(B, Hq, Hkv, D, block_size, BOUND, G.SPLIT_BALANCED)[0], dtype=torch.uint8, device="cuda")
    for step in (True, False):
        rows = W.all_token_rows(case, include_new=not step)
        dk, dv = (torch.full(kc8.shape, 0x7F, dtype=torch.uint8, device="cuda") for _ in range(2))
        if len(rows[2]):
            G.reshape_and_cache_fp8(U.to_dev(rows[0], dtype), U.to_dev(rows[1], dtype), dk, dv, torch.from_numpy(rows[2]).cuda(), k_scale, v_scale)
        dev.out.fill_(float("nan"))
        ws.fill_(0xFF)
        if step:
            G.decode_step_fp8(dev.out, dev.q, dev.k_new, dev.v_new, dk, dv, dev.block_tables, dev.context_lens, dev.slopes, float(case.scale),
                              k_scale, v_scale, BOUND, ws)
        else:
            G.paged_attention_fp8(dev.out, dev.q, dk, dv, dev.block_tables, dev.context_lens, dev.slopes, float(case.scale), k_scale, v_scale,
                                  BOUND, ws)
        torch.cuda.synchronize()
        dev.check_canaries()
        assert np.array_equal(dk.cpu().numpy(), kc8) and np.array_equal(dv.cpu().numpy(), vc8)
        assert U.max_abs_err(U.to_host(dev.out), ref, dtype) <= U.TOL[dtype]
