"""GPU parity of decode over 8-bit caches where a wave may take two tiles at a time (head_dim 128, a bound under which there may be many
tiles; the device chooses by the tiles that there are): units of one, few and many tiles, odd ones among them, sequences of one
token, several pieces to a unit, in either way of taking them; and what a wide bound costs short sequences."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu
BOUND = 4096                        # 16 sequences x 8 KV heads x 256 tiles: 32 tiles to each of 1 024 units


def pairs_from(B, Hq, Hkv, bound, cus):
    """The tiles from which a launch's units are taken two tiles at a time (decode_split.hpp's rule); 0: never."""
    group = Hq // Hkv
    segments = B * Hkv * (group // max(h for h in range(1, 17) if group % h == 0))
    if segments * -(-bound // 16) < 32 * 4 * cus:
        return 0
    return min((18 if B * Hq <= 4 * cus else 2) * 4 * cus + 160 * max(segments - cus, 0), 2**31 - 1)


# (the first four: tile by tile; the last: in pairs)
@pytest.mark.parametrize("lo,hi", [(1, 5), (1, 70), (15, 700), (1, 4096), (4081, 4096)])
@pytest.mark.parametrize("Hq,block_size", [(8, 16), (32, 64)])
@pytest.mark.parametrize("dtype", [W.BF16, W.F16])
def test_two_tiles_at_a_time(U, oracle, dtype, Hq, block_size, lo, hi):
    import torch
    import oracle as O
    import pins_e4m3
    import paper_2505_02351_amd as G
    B, Hkv, D, k_scale, v_scale = 16, 8, 128, 0.0125, 0.03
    tiles = pairs_from(B, Hq, Hkv, BOUND, torch.cuda.get_device_properties(0).multi_processor_count)
    assert tiles > 0 and (lo < 4000 or B * Hkv * (lo // 16) >= tiles)
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


# (sequences, heads, KV heads, longest, bound): more sequences than lanes, one, two and five chunks of heads; in pairs (units of two or three
# tiles, many pieces of one) and, short, tile by tile
@pytest.mark.parametrize("B,Hq,Hkv,hi,bound,pairs", [
    (66, 32, 2, 700, 4096, True), (66, 32, 2, 100, 4096, False), (260, 16, 1, 400, 2048, True), (260, 16, 1, 90, 2048, False),
    (64, 32, 4, 300, 2048, True), (17, 80, 1, 1500, 8192, True), (32, 64, 8, 500, 2048, True), (32, 64, 8, 30, 2048, False)])
@pytest.mark.parametrize("dtype,alibi,heads", [(W.BF16, True, True), (W.F16, False, False)])
def test_many_sequences_and_empty_ones(U, oracle, dtype, alibi, heads, B, Hq, Hkv, hi, bound, pairs):
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    D, bs = 128, 16
    cfg = W.small_config(name="many", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=bs,
                         num_blocks=B * -(-hi // bs) + 7, ctx_lo=1, ctx_hi=hi, seed=hi + B)
    case = W.make_case(cfg)
    rng = np.random.default_rng(B + hi)
    if heads:
        k_scales, v_scales = ((0.0125 * np.exp2(rng.integers(-2, 3, size=Hkv))).astype(np.float32) for _ in range(2))
    else:
        k_scales, v_scales = (np.full(Hkv, x, np.float32) for x in (0.0125, 0.03))
    rows = W.all_token_rows(case)
    kc8, vc8 = (np.full((cfg.num_blocks, Hkv, bs, D), 0x7F, np.uint8) for _ in range(2))
    O.reshape_and_cache_e4m3_heads(*rows[:2], kc8, vc8, rows[2], k_scales, v_scales, dtype)
    lens = case.context_lens.copy()
    empty = [0, 5, 6, B - 1]
    lens[empty] = 0
    tiles = Hkv * max(Hq // Hkv // 16, 1) * int(sum(-(-(n - 1) // 16) for n in lens if n))      # (groups of up to 16, or of 80)
    line = pairs_from(B, Hq, Hkv, bound, torch.cuda.get_device_properties(0).multi_processor_count)
    assert line > 0 and (tiles >= line) == pairs, (tiles, line)
    some = [(b, h) for b in (0, 1, 6, B // 2, B - 2, B - 1) for h in range(Hq)]
    slopes = case.slopes if alibi else None
    ref = O.paged_attention_e4m3_heads(case.q, kc8, vc8, case.block_tables, lens, slopes, case.scale, k_scales, v_scales, dtype, rows=some)
    case.block_tables = np.pad(case.block_tables, ((0, 0), (0, bound // bs - case.block_tables.shape[1])), constant_values=-1)
    dev = U.DevCase(case)
    dlens, sl = torch.from_numpy(lens).cuda(), dev.slopes if alibi else None
    ks, vs = (torch.from_numpy(x).cuda() for x in (k_scales, v_scales))
    ws = torch.empty(G.paged_attention_workspace_bytes(B, Hq, Hkv, D, bs, bound, G.SPLIT_BALANCED)[0], dtype=torch.uint8, device="cuda")
    for step in (True, False):
        dk, dv = (torch.from_numpy(x).cuda() for x in (kc8, vc8))
        slots = case.slot_mapping
        if step:                                # the step has to put the new rows' codes in, but for the empty sequences'
            for c in (dk, dv):
                c[torch.from_numpy(slots // bs).cuda(), :, torch.from_numpy(slots % bs).cuda()] = 0x7F
        dev.out.fill_(float("nan"))
        ws.fill_(0xFF)
        args = (dev.block_tables, dlens, sl, float(case.scale)) + ((ks, vs) if heads else (float(k_scales[0]), float(v_scales[0]))) + (bound, ws)
        if step:
            (G.decode_step_fp8_heads if heads else G.decode_step_fp8)(dev.out, dev.q, dev.k_new, dev.v_new, dk, dv, *args)
        else:
            (G.paged_attention_fp8_heads if heads else G.paged_attention_fp8)(dev.out, dev.q, dk, dv, *args)
        torch.cuda.synchronize()
        dev.check_canaries()
        for got, want in ((dk, kc8), (dv, vc8)):
            want = want.copy()
            if step:
                want[slots[empty] // bs, :, slots[empty] % bs] = 0x7F
            assert np.array_equal(got.cpu().numpy(), want)
        out = U.to_host(dev.out)
        assert np.isfinite(W.from_bits(out, dtype)).all() and (out[empty] == 0).all()
        U.check_scaled(np.stack([out[b, h] for b, h in some]), ref, dtype, f"{B} sequences, step {step}")


# (sequences, KV heads, lengths, a bound below the line and the next block's): a bound at which the device may choose pairs used to
# take them whatever the lengths: 1.31 and 1.54 of the time; 0.98 to 1.01 and 1.02 to 1.04 since it compares the tiles that there are
@pytest.mark.parametrize("B,lo,hi,below,above", [(200, 31, 255, 320, 336), (200, 15, 127, 320, 336)])
def test_short_sequences_do_not_pay_for_a_wide_bound(U, B, lo, hi, below, above):
    import torch
    import paper_2505_02351_amd as G
    from test_gpu_decode_unsplit_step import microseconds
    Hq, Hkv, D, bs = 32, 8, 128, 16
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert pairs_from(B, Hq, Hkv, below, cus) == 0 < pairs_from(B, Hq, Hkv, above, cus)
    rng = np.random.default_rng(B)
    lens = torch.from_numpy(rng.integers(lo, hi + 1, B).astype(np.int32)).cuda()
    blocks = -(-hi // bs)
    table = torch.zeros(B, above // bs, dtype=torch.int32, device="cuda")
    table[:, :blocks] = torch.randperm(B * blocks, device="cuda").to(torch.int32).view(B, blocks)
    q, k, v = (torch.randn(B, h, D, device="cuda", dtype=torch.bfloat16) for h in (Hq, Hkv, Hkv))
    kc, vc = (torch.randint(0, 0x70, (B * blocks, Hkv, bs, D), device="cuda", dtype=torch.uint8) for _ in range(2))
    out = torch.empty_like(q)
    slopes = torch.exp2(-8.0 * torch.arange(1, Hq + 1, device="cuda") / Hq)
    ws = torch.empty(G.paged_attention_workspace_bytes(B, Hq, Hkv, D, bs, above, G.SPLIT_BALANCED)[0], dtype=torch.uint8, device="cuda")

    def us(bound):
        def call():
            G.decode_step_fp8(out, q, k, v, kc, vc, table, lens, slopes, D ** -0.5, 0.01, 0.01, bound, ws)
        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                call()
        return microseconds(graph.replay, reps=1, runs=15) / 20
    narrow, wide = us(below), us(above)
    assert wide <= 1.08 * narrow, (wide, narrow)
