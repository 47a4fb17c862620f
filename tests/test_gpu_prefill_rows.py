"""GPU parity of how the tiled prefill kernel takes its query rows in, hands its output rows out, and stores a step's new
K/V rows: whole rows at a time, for groups that do and do not fill a workgroup's rows, in every workgroup shape."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U, oracle_filled  # noqa: F401  (U: a fixture)
from test_gpu_prefill_walk import launch_shape

pytestmark = pytest.mark.gpu


# (sequences, heads, KV heads, new tokens): groups of 1 (128 or 256 tokens to a workgroup: more new rows than its threads take
# in one go), 3 (a quarter of the rows are nobody's), 4, 16; a last token tile of one token, of all but one, and full
@pytest.mark.parametrize("B,Hq,Hkv,q_len,shape", [
    (1, 2, 2, 1, "two"), (1, 2, 2, 129, "two"), (2, 6, 2, 33, "two"), (2, 16, 1, 9, "two"),
    (20, 16, 16, 129, "4"), (44, 12, 4, 63, "4"), (40, 32, 8, 33, "4"), (130, 32, 2, 8, "4"),
    (16, 32, 32, 257, "8"), (64, 24, 8, 65, "8"), (66, 32, 8, 63, "8"), (260, 32, 2, 15, "8")])
@pytest.mark.parametrize("ctx,alibi", [(0, True), (21, False), (530, True)])   # (16 tiles or more with slopes: a wave's rows are one head's)
@pytest.mark.parametrize("dtype,D", [(W.BF16, 128), (W.F16, 64)])
def test_rows_in_and_out(U, oracle, dtype, D, ctx, alibi, B, Hq, Hkv, q_len, shape):
    L = ctx + q_len
    # (256 rows: with slopes, head_dim 128)
    assert launch_shape(B, Hq, Hkv, q_len, D=D, slopes=alibi, longest=-(-L // 16) * 16)[0] == (shape if alibi and D == 128 or shape == "two" else "4")
    cfg = W.small_config(name="rows", kind="prefill", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D,
                         block_size=16, num_blocks=B * -(-L // 16) + 3, ctx_lo=L, ctx_hi=L, q_len=q_len, seed=31 + B + q_len)
    case = W.make_case(cfg)
    if not alibi:
        case.slopes = None
    dev = U.DevCase(case)
    dev.out.fill_(float("nan"))
    step = dev.prefill_step()                   # (canaries on either side of the output are checked in there)
    kc, vc = oracle_filled(oracle, case)
    assert (U.to_host(dev.k_cache) == kc).all() and (U.to_host(dev.v_cache) == vc).all()
    some = min(B, 3)                            # the oracle's time: the first sequences and the last
    for first, last in {(0, some), (B - 1, B)}:
        cu = case.cu_q_lens[first:last + 1]
        rows = slice(cu[0], cu[-1])
        ref = oracle.paged_prefill(case.q[rows], kc, vc, case.block_tables[first:last], case.context_lens[first:last],
                                   cu - cu[0], case.slopes, case.scale, dtype)
        U.check_scaled(step[rows], ref, dtype, f"prefill step, sequences {first}-{last}")
    assert np.isfinite(W.from_bits(step, dtype)).all()
    assert (dev.prefill() == step).all()        # rows written by a call of its own: the same bits


@pytest.mark.parametrize("bound", [2047, 2048])                 # far above the lengths
@pytest.mark.parametrize("dtype,D", [(W.BF16, 128), (W.F16, 128), (W.BF16, 64)])
@pytest.mark.parametrize("alibi", [True, False])
def test_whole_prompts_under_a_loose_bound(U, dtype, D, alibi, bound):
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    B, Hq, Hkv, q_len = 2, 32, 8, 173
    assert launch_shape(B, Hq, Hkv, bound, True, D=D, slopes=alibi, longest=bound)[0] == "4"
    cfg = W.small_config(name="long", kind="prefill", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D,
                         block_size=16, num_blocks=B * 11 + 3, ctx_lo=q_len, ctx_hi=q_len, q_len=q_len, seed=bound)
    case = W.make_case(cfg)
    if not alibi:
        case.slopes = None
    case.block_tables = np.pad(case.block_tables, ((0, 0), (0, 2048 // 16 - case.block_tables.shape[1])), constant_values=-1)
    dev = U.DevCase(case)
    dev.out.fill_(float("nan"))
    G.prompt_prefill(dev.out, dev.q, dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_tables, dev.cu_q_lens,
                     dev.slopes, float(case.scale), bound)
    torch.cuda.synchronize()
    dev.check_canaries()
    ref = O.prompt_attention(case.q, case.k_new, case.v_new, case.cu_q_lens, case.slopes, case.scale, dtype)
    U.check_scaled(U.to_host(dev.out), ref, dtype, f"whole prompts, at most {bound} tokens")
