"""GPU parity where a prefill tile goes to LDS without passing through registers: walks over more blocks than a lane read
reaches without reading the table anew, whole prompts under a bound for which they take 256-row workgroups, and rows of the inputs further
apart than a lane's offset reaches."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


# (sequences, heads, KV heads): two key groups, 128 and 256 rows (slopes, head_dim 128; 128 rows without); 64 blocks of a table are read at once
@pytest.mark.parametrize("B,Hq,Hkv", [(2, 8, 2), (70, 8, 2), (56, 8, 8)])
@pytest.mark.parametrize("ctx", [1023 + 16, 1024 + 17, 2111])
@pytest.mark.parametrize("dtype,D,alibi", [(W.BF16, 128, True), (W.F16, 128, False), (W.BF16, 64, True)])
def test_walks_over_many_blocks(U, oracle, dtype, D, alibi, ctx, B, Hq, Hkv):
    import torch
    import paper_2505_02351_amd as G
    bs, q_len, rng = 16, 70, np.random.default_rng(ctx + B)
    blocks, own = -(-ctx // bs), 2                              # two sequences' blocks; the others read theirs
    kc, vc = (W.to_bits(rng.standard_normal((own * blocks + 3, Hkv, bs, D)).astype(np.float32), dtype) for _ in range(2))
    order = rng.permutation(own * blocks + 3)[:own * blocks].astype(np.int32).reshape(own, blocks)
    tables = np.ascontiguousarray(order[np.arange(B) % own])
    lens, cu = np.full(B, ctx, np.int32), (np.arange(B + 1) * q_len).astype(np.int32)
    q = W.to_bits(rng.standard_normal((B * q_len, Hq, D)).astype(np.float32), dtype)
    slopes = (2.0 ** -(8 + np.arange(Hq) / Hq)).astype(np.float32) if alibi else None      # (nothing is out of the question)
    scale = 1 / np.sqrt(np.float32(D))
    dev = [U.to_dev(x, dtype) for x in (q, kc, vc)]
    out = torch.full_like(dev[0], float("nan"))
    G.paged_prefill(out, *dev, *(torch.from_numpy(x).cuda() for x in (tables, lens, cu)),
                    None if slopes is None else torch.from_numpy(slopes).cuda(), float(scale), q_len)
    torch.cuda.synchronize()
    got = U.to_host(out)
    assert np.isfinite(W.from_bits(got, dtype)).all()
    for b in (0, B - 1):
        rows = slice(cu[b], cu[b + 1])
        ref = oracle.paged_prefill(q[rows], kc, vc, tables[b:b + 1], lens[b:b + 1], cu[:2], slopes, scale, dtype)
        U.check_scaled(got[rows], ref, dtype, f"sequence {b}")


@pytest.mark.parametrize("q_len", [1, 33, 257, 705])            # the last tile of one key, one more than a tile; several query tiles
@pytest.mark.parametrize("dtype", [W.BF16, W.F16])
def test_whole_prompts_in_256_rows(U, dtype, q_len):
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    B, Hq, Hkv, bound = 54, 8, 8, 3100                          # 432 x 13 workgroups of 256 rows under the bound
    cfg = W.small_config(name="prompts", kind="prefill", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=128,
                         block_size=16, num_blocks=B * -(-q_len // 16) + 3, ctx_lo=q_len, ctx_hi=q_len, q_len=q_len, seed=q_len)
    case = W.make_case(cfg)
    case.block_tables = np.pad(case.block_tables, ((0, 0), (0, -(-bound // 16) - case.block_tables.shape[1])), constant_values=-1)
    dev = U.DevCase(case)
    dev.out.fill_(float("nan"))
    G.prompt_prefill(dev.out, dev.q, dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_tables, dev.cu_q_lens,
                     dev.slopes, float(case.scale), bound)
    torch.cuda.synchronize()
    dev.check_canaries()
    got = U.to_host(dev.out)
    assert np.isfinite(W.from_bits(got, dtype)).all()
    for first, last in ((0, 2), (B - 1, B)):
        cu = case.cu_q_lens[first:last + 1]
        rows = slice(cu[0], cu[-1])
        ref = O.prompt_attention(case.q[rows], case.k_new[rows], case.v_new[rows], cu - cu[0], case.slopes, case.scale, dtype)
        U.check_scaled(got[rows], ref, dtype, f"prompts {first}-{last}")


# elements from token to token: the most that lane offsets of 32 bits reach over a load's rows, and the next
@pytest.mark.parametrize("stride", [2**28 - 8, 2**28])
@pytest.mark.parametrize("dtype,D,Hq,Hkv", [(W.BF16, 128, 4, 2), (W.F16, 64, 4, 1)])
def test_rows_far_apart(U, dtype, D, Hq, Hkv, stride):
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    n = 97                                      # four tiles: those behind the first two have lane offsets, or lane addresses
    cfg = W.small_config(name="apart", kind="prefill", dtype=dtype, batch=1, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=16, num_blocks=8,
                         ctx_lo=n, ctx_hi=n, q_len=n, seed=D)
    case = W.make_case(cfg)
    dev = U.DevCase(case)
    row = Hkv * D
    pool = torch.empty((n - 1) * stride + 2 * row, dtype=dev.q.dtype, device="cuda")             # 48 GiB, of which a few rows are touched
    k, v = (pool[at:].as_strided((n, Hkv, D), (stride, D, 1)) for at in (0, row))
    k.copy_(dev.k_new), v.copy_(dev.v_new)
    dev.out.fill_(float("nan"))
    G.prompt_prefill(dev.out, dev.q, k, v, dev.k_cache, dev.v_cache, dev.block_tables, dev.cu_q_lens, dev.slopes, float(case.scale), n)
    torch.cuda.synchronize()
    dev.check_canaries()
    got = U.to_host(dev.out)
    del pool, k, v
    torch.cuda.empty_cache()
    U.check_scaled(got, O.prompt_attention(case.q, case.k_new, case.v_new, case.cu_q_lens, case.slopes, case.scale, dtype), dtype, f"stride {stride}")
    kc, vc = (x.copy() for x in (case.k_cache, case.v_cache))
    O.reshape_and_cache(case.k_new, case.v_new, kc, vc, case.slot_mapping)
    assert (U.to_host(dev.k_cache) == kc).all() and (U.to_host(dev.v_cache) == vc).all()
