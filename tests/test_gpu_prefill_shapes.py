"""GPU parity where the width of the block tables, or a bound on the chunks, alone makes a prefill workgroup's rows 256; and times of the shapes
against a kernel of the same library that always has 128."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U, oracle_filled  # noqa: F401  (a fixture)
from test_gpu_prefill_walk import launch_shape

pytestmark = pytest.mark.gpu


def at_both_ends(U, oracle, case, got, dtype, cu, n=3, tag=""):
    kc, vc = oracle_filled(oracle, case)
    B = len(cu) - 1
    for first, last in {(0, min(B, n)), (max(B - n, 0), B)}:
        c = cu[first:last + 1]
        rows = slice(c[0], c[-1])
        ref = oracle.paged_prefill(case.q[rows], kc, vc, case.block_tables[first:last], case.context_lens[first:last], c - c[0], case.slopes, case.scale,
                                   dtype)
        U.check_scaled(got[rows], ref, dtype, f"{tag}, sequences {first}-{last}")


# no slopes: what the tables hold is more than the last-level cache keeps, or the bound on a chunk more than 2 048 tokens
@pytest.mark.parametrize("B,Hq,Hkv,q_len,wide,bound", [(64, 8, 8, 150, 1300, None), (66, 8, 8, 300, 1200, None), (64, 8, 2, 9, 208, 2100)])
@pytest.mark.parametrize("dtype", [W.BF16, W.F16])
def test_256_rows_without_slopes(U, oracle, dtype, B, Hq, Hkv, q_len, wide, bound):
    import torch
    import paper_2505_02351_amd as G
    ctx, D = q_len + 40, 128
    assert launch_shape(B, Hq, Hkv, bound or q_len, slopes=False, longest=wide)[0] == "8"
    cfg = W.small_config(name="far", kind="prefill", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=16,
                         num_blocks=B * -(-ctx // 16) + 3, ctx_lo=q_len, ctx_hi=ctx, q_len=q_len, seed=B + q_len)
    case = W.make_case(cfg)
    case.slopes = None
    more = -(-wide // 16) - case.block_tables.shape[1]
    case.block_tables = np.pad(case.block_tables, ((0, 0), (0, more)), constant_values=-1)
    dev = U.DevCase(case)
    dev.out.fill_(float("nan"))
    G.prefill_step(dev.out, dev.q, dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_tables, dev.context_lens, dev.cu_q_lens, None,
                   float(case.scale), bound or case.max_q_len)
    torch.cuda.synchronize()
    dev.check_canaries()
    at_both_ends(U, oracle, case, U.to_host(dev.out), dtype, case.cu_q_lens, tag="256 rows")


def timed(B, Hq, Hkv, D, new, ctx, slopes, dtype):
    """GPU time of plain prefill over 2-byte and over 8-bit caches, and under a window that hides nothing."""
    import torch
    import paper_2505_02351_amd as G
    from test_gpu_decode_unsplit_step import microseconds
    bs, blocks = 32, -(-(ctx + new) // 32)
    gen = torch.Generator("cuda").manual_seed(4)
    q = torch.randn(B * new, Hq, D, generator=gen, device="cuda").to(dtype)
    kc, vc = (torch.randn(B * blocks, Hkv, bs, D, generator=gen, device="cuda", dtype=dtype) for _ in range(2))
    table = torch.randperm(B * blocks, generator=gen, device="cuda").to(torch.int32).view(B, blocks)
    lens = torch.full((B,), ctx + new, dtype=torch.int32, device="cuda")
    cu = torch.arange(0, B * new + 1, new, dtype=torch.int32, device="cuda")
    sl = torch.exp2(-8.0 * torch.arange(1, Hq + 1, device="cuda") / Hq) if slopes else None
    out = torch.empty_like(q)
    plain = microseconds(lambda: G.paged_prefill(out, q, kc, vc, table, lens, cu, sl, D ** -0.5, new))
    windowed = microseconds(lambda: G.paged_prefill_window(out, q, kc, vc, table, lens, cu, sl, D ** -0.5, 32768, new))
    k8, v8 = ((torch.randn(B * blocks, Hkv, bs, D, generator=gen, device="cuda", dtype=dtype) * 80).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
              for _ in range(2))
    return plain, microseconds(lambda: G.paged_prefill_fp8(out, q, k8, v8, table, lens, cu, sl, D ** -0.5, 0.0125, 0.0125, new)), windowed


@pytest.mark.parametrize("B,Hq,Hkv,new,ctx,slopes,limit", [(30, 16, 16, 2, 1000, True, 1.12), (30, 16, 16, 100, 1000, True, 1.15), (100, 16, 16, 131, 1000, False, 0.93),
                                                             (40, 16, 16, 500, 1000, False, 0.95)])
def test_workgroups_are_as_wide_as_it_pays(U, B, Hq, Hkv, new, ctx, slopes, limit):
    """Against the windowed kernel, whose workgroups always have 128 rows: 1.24, 1.37, 0.99 and 1.03 of its time when 480 half empty
    workgroups had 256 rows and none had them without slopes; 1.00, 0.97, 0.85 and 0.89."""
    import torch
    plain, _, windowed = timed(B, Hq, Hkv, 128, new, ctx, slopes, torch.bfloat16)
    assert plain <= limit * windowed, (plain, windowed)
