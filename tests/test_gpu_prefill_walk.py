"""GPU parity of how the tiled prefill kernel ends, orders and shares out its walks: the rest of a walk that
is judged at once from the keys' norms, ragged launches ordered by length, walks shared by two key groups."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U, fp8_caches, oracle_filled  # noqa: F401  (U: a fixture)

pytestmark = pytest.mark.gpu


def row_tiles(Hq, Hkv, max_q_len, rows):
    """Workgroups of that many rows to a unit."""
    group = Hq // Hkv
    gh = max(h for h in range(1, 17) if group % h == 0)
    return -(-max_q_len // (rows // (1 << (gh - 1).bit_length())))


def units(batch, Hq, Hkv):
    group = Hq // Hkv
    return -(-batch * Hkv * (group // max(h for h in range(1, 17) if group % h == 0)) // 8) * 8


def cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def launch_shape(batch, Hq, Hkv, max_q_len, whole_prompt=False, D=128, slopes=True, kv8=False, window=0, longest=0):
    """The workgroup shape that a prefill launch takes on this card (prefill_shape.hpp's rules): "two" key groups of four
    waves, "4" waves, or "8" waves; and its query tiles.  longest: tokens that a block table holds."""
    tiles4, tiles8, u = row_tiles(Hq, Hkv, max_q_len, 128), row_tiles(Hq, Hkv, max_q_len, 256), units(batch, Hq, Hkv)
    if window:
        return "4", tiles4
    if u * tiles4 <= cus():
        return "two", tiles4
    if kv8:
        wide = u * tiles8 >= 2 * cus()
    else:
        far = 4 * batch * longest * Hkv * D >= 320000000
        if whole_prompt:
            wide = u * tiles8 > 5 * cus() and (max_q_len > 3072 if slopes else far)
        elif slopes:
            wide = 4 * u * tiles8 >= (7 if tiles8 > 1 else 8) * cus()
        else:
            wide = u * tiles8 >= 2 * cus() and (tiles4 > tiles8 and far or max_q_len > 2048)
        wide = wide and D == 128
    return ("8", tiles8) if wide else ("4", tiles4)


def launch_deep(batch, Hq, Hkv, max_q_len, slopes=True, window=0, longest=0):
    """Whether a launch over 2-byte caches asks for its tiles two steps ahead."""
    tiles4 = row_tiles(Hq, Hkv, max_q_len, 128)
    seen = min(longest, window + max_q_len) if window else longest
    if tiles4 > 2:
        return slopes and not window and tiles4 <= 16 and seen >= 4096
    return units(batch, Hq, Hkv) * tiles4 > cus() or seen >= (512 if tiles4 == 1 else 1000)


LONGEST = 1600          # tokens that a launch's longest possible walk must have for its kernel to look at the rest of walks (48 tiles)


def widen(case, longest=LONGEST):
    """Block tables as wide as a serving program's, for sequences of up to `longest` tokens: what the launch goes by."""
    bs = case.cfg.block_size
    more = -(-longest // bs) - case.block_tables.shape[1]
    case.block_tables = np.pad(case.block_tables, ((0, 0), (0, max(more, 0))), constant_values=-1)
    assert case.block_tables.shape[1] * bs >= longest


def outlier_case(dtype, D, q_len, t0, slope, like, ctx=705, batch=2, seed=1, heads=(8, 2), block_size=16):
    """Steep slopes, under which every key far back is out of the question - except the one at t0 of
    sequence 0, whose K row points along the last query (of head 1): its score outweighs its bias by 3."""
    cfg = W.small_config(name="outlier", kind="prefill", dtype=dtype, batch=batch, num_heads=heads[0], num_kv_heads=heads[1],
                         head_dim=D, block_size=block_size, num_blocks=batch * -(-ctx // block_size) + 3, ctx_lo=ctx, ctx_hi=ctx, q_len=q_len, seed=seed)
    case = W.make_case(cfg, slopes=np.full(heads[0], slope, np.float32))
    g = 1 * heads[1] // heads[0]                # head 1's KV head
    q = W.from_bits(case.q[case.cu_q_lens[1] - 1, 1], dtype)
    want = slope * (ctx - 1 - t0) + 3.0
    row = np.sign(q) * 5.6 if like == "sign" else q * (want / (float(case.scale) * float(q @ q)))
    assert float(case.scale) * float(row @ q) > want - 0.5
    bits = W.to_bits(row.astype(np.float32), dtype)
    new = t0 - (ctx - q_len)
    if new >= 0:
        case.k_new[new, g] = bits
    else:
        case.k_cache[case.block_tables[0, t0 // block_size], g, t0 % block_size] = bits
    widen(case)
    return case


@pytest.mark.parametrize("t0", [0, 15, 16, 333, 511])
@pytest.mark.parametrize("dtype,D", [(W.BF16, 128), (W.F16, 64)])
@pytest.mark.parametrize("batch,heads,q_len,shape", [(2, (8, 2), 24, "two"), (70, (8, 2), 70, "4"), (64, (8, 8), 70, "8")])   # ("8": head_dim 128)
@pytest.mark.parametrize("block_size", [16, 64])
def test_a_far_key_that_matters_is_not_judged_away(U, oracle, block_size, batch, heads, q_len, shape, dtype, D, t0):
    assert launch_shape(batch, *heads, q_len, D=D)[0] == (shape if D == 128 or shape == "two" else "4")
    case = outlier_case(dtype, D, q_len, t0, 0.25, "q", batch=batch, heads=heads, block_size=block_size)
    dev = U.DevCase(case)
    step = dev.prefill_step()
    kc, vc = oracle_filled(oracle, case)
    rows = slice(None, case.cu_q_lens[2])       # sequences 0 and 1
    ref = oracle.paged_prefill(case.q[rows], kc, vc, case.block_tables[:2], case.context_lens[:2], case.cu_q_lens[:3],
                               case.slopes, case.scale, dtype)
    U.check_scaled(step[rows], ref, dtype, f"prefill step, outlier at {t0}")
    U.check_scaled(dev.prefill()[rows], ref, dtype, f"paged prefill, outlier at {t0}")


@pytest.mark.parametrize("t0", [0, 16, 511, 640])
@pytest.mark.parametrize("batch,heads,shape,bound", [(2, (8, 8), "two", LONGEST), (6, (8, 2), "4", LONGEST), (54, (8, 8), "4", LONGEST),
                                                     (54, (8, 8), "8", 3100)])      # ("8": head_dim 128)
@pytest.mark.parametrize("dtype,D", [(W.BF16, 128), (W.F16, 64)])
def test_a_far_key_of_a_whole_prompt(U, oracle, dtype, D, batch, heads, shape, bound, t0):
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    assert launch_shape(batch, *heads, bound, True, D=D)[0] == (shape if D == 128 or shape == "two" else "4")
    case = outlier_case(dtype, D, 705, t0, 0.25, "q", batch=batch, heads=heads)
    widen(case, bound)
    dev = U.DevCase(case)
    G.prompt_prefill(dev.out, dev.q, dev.k_new, dev.v_new, dev.k_cache, dev.v_cache, dev.block_tables, dev.cu_q_lens,
                     dev.slopes, float(case.scale), bound)
    torch.cuda.synchronize()
    dev.check_canaries()
    rows = slice(None, case.cu_q_lens[2])       # sequences 0 and 1
    ref = O.prompt_attention(case.q[rows], case.k_new[rows], case.v_new[rows], case.cu_q_lens[:3], case.slopes, case.scale, dtype)
    U.check_scaled(U.to_host(dev.out)[rows], ref, dtype, f"whole prompt, outlier at {t0}")


@pytest.mark.parametrize("t0", [0, 16, 511])
@pytest.mark.parametrize("batch,heads,q_len,shape", [(2, (8, 2), 24, "two"), (70, (8, 2), 70, "4"), (64, (8, 8), 24, "8")])
@pytest.mark.parametrize("D", [128, 64])
def test_a_far_key_of_an_8_bit_cache(U, oracle, D, batch, heads, q_len, shape, t0):
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    assert launch_shape(batch, *heads, q_len, D=D, kv8=True)[0] == shape
    case = outlier_case(W.BF16, D, q_len, t0, 1 / 16 if D == 128 else 1 / 32, "sign", batch=batch, heads=heads)
    kc8, vc8, dk, dv = fp8_caches(U, case, 0.0125, 0.02)
    qd = U.to_dev(case.q, W.BF16)
    out = torch.full_like(qd, float("nan"))
    G.paged_prefill_fp8(out, qd, dk, dv, torch.from_numpy(case.block_tables).cuda(),
                        torch.from_numpy(case.context_lens).cuda(), torch.from_numpy(case.cu_q_lens).cuda(),
                        torch.from_numpy(case.slopes).cuda(), float(case.scale), 0.0125, 0.02, case.max_q_len)
    torch.cuda.synchronize()
    rows = slice(None, case.cu_q_lens[2])       # sequences 0 and 1
    ref = O.paged_prefill_e4m3(case.q[rows], kc8, vc8, case.block_tables[:2], case.context_lens[:2], case.cu_q_lens[:3],
                               case.slopes, case.scale, 0.0125, 0.02, W.BF16)
    U.check_scaled(U.to_host(out)[rows], ref, W.BF16, f"E4M3 caches, outlier at {t0}")


@pytest.mark.parametrize("t0", [None, 5, 1000, 2000])
@pytest.mark.parametrize("block_size", [16, 32])
@pytest.mark.parametrize("batch,heads,D,shape", [(2, (8, 2), 64, "two"), (64, (8, 8), 64, "4"), (64, (8, 8), 128, "8")])
def test_a_far_key_under_a_negative_slope(U, oracle, batch, heads, D, shape, block_size, t0):
    """Biases that grow with the distance, by 20 over the context; near keys whose scores lie 60 above the others' end the
    walk all the same - unless one far key's score makes up for what its bias leaves."""
    ctx, q_len, slope = 2616, 24, -2.0 ** -7
    assert launch_shape(batch, *heads, q_len, D=D)[0] == shape
    cfg = W.small_config(name="negative", kind="prefill", dtype=W.BF16, batch=batch, num_heads=heads[0], num_kv_heads=heads[1],
                         head_dim=D, block_size=block_size, num_blocks=batch * -(-ctx // block_size), ctx_lo=ctx, ctx_hi=ctx,
                         q_len=q_len, seed=6)
    case = W.make_case(cfg, slopes=np.full(heads[0], slope, np.float32))
    pos0, u = ctx - q_len, np.full(D, D ** -0.5, np.float32)

    def put(b, t, score):
        row = W.to_bits(u * np.float32(score / case.scale), W.BF16)
        if t >= pos0:
            case.k_new[b * q_len + t - pos0] = row
        else:
            case.k_cache[case.block_tables[b, t // block_size], :, t % block_size] = row
    case.q[:] = W.to_bits(u, W.BF16)
    case.k_cache[:] = case.k_new[:] = 0
    for b in range(batch):
        for t in (pos0, pos0 - 4, pos0 - 8):
            put(b, t, 60.0)
    if t0 is not None:
        put(0, t0, 60.0 + 2.0 + slope * (ctx - t0))
    dev = U.DevCase(case)
    step = dev.prefill_step()
    kc, vc = oracle_filled(oracle, case)
    rows = slice(None, case.cu_q_lens[2])
    ref = oracle.paged_prefill(case.q[rows], kc, vc, case.block_tables[:2], case.context_lens[:2], case.cu_q_lens[:3],
                               case.slopes, case.scale, W.BF16)
    U.check_scaled(step[rows], ref, W.BF16, f"negative slope, outlier at {t0}", max_exempt=1.0)


@pytest.mark.parametrize("B,Hq,Hkv,D,shape", [(2, 8, 2, 128, "two"), (64, 8, 8, 64, "4"), (64, 8, 8, 128, "8")])
def test_half_a_rows_sum_does_not_judge_the_other_halfs_keys(U, oracle, B, Hq, Hkv, D, shape):
    """A row's sum is held by two lanes, of keys 8i .. 8i + 3 and 8i + 4 .. 8i + 7.  Two near keys of the first kind weigh
    2^23 times the others, so the far keys lie below 2^-24 of the whole sum, but not of the second lane's half of it:
    a tile of them is kept, and so must be the rest of the walk (their values are large: without them the output is
    off by 0.4 or more)."""
    ctx, q_len = 2616, 24
    assert launch_shape(B, Hq, Hkv, q_len, D=D)[0] == shape
    cfg = W.small_config(name="halves", kind="prefill", dtype=W.BF16, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D,
                         block_size=16, num_blocks=B * 164, ctx_lo=ctx, ctx_hi=ctx, q_len=q_len, seed=3)
    case = W.make_case(cfg, slopes=np.full(Hq, 2.0 ** -9, np.float32))
    pos0, u = ctx - q_len, np.full(D, D ** -0.5, np.float32)
    case.q[:] = W.to_bits(u, W.BF16)
    case.k_cache[:] = case.k_new[:] = 0
    loud = W.to_bits(u * np.float32(23 * np.log(2) / case.scale), W.BF16)
    for b in range(B):                      # positions 2 592 and 2 584: in the first tile of either key group
        case.k_new[b * q_len] = loud
        case.k_cache[case.block_tables[b, (pos0 - 8) // 16], :, (pos0 - 8) % 16] = loud
        for t in range(0, pos0 - 400, 16):
            case.v_cache[case.block_tables[b, t // 16]] = W.to_bits(np.float32(3e4), W.BF16)
    dev = U.DevCase(case)
    step = dev.prefill_step()
    kc, vc = oracle_filled(oracle, case)
    rows = slice(None, case.cu_q_lens[2])
    ref = oracle.paged_prefill(case.q[rows], kc, vc, case.block_tables[:2], case.context_lens[:2], case.cu_q_lens[:3],
                               case.slopes, case.scale, W.BF16)
    U.check_scaled(step[rows], ref, W.BF16, "halves", max_exempt=1.0)


@pytest.mark.parametrize("B,Hq,Hkv,D,shape", [(2, 8, 2, 128, "two"), (64, 8, 8, 64, "4"), (64, 8, 8, 128, "8")])
def test_a_key_whose_norm_overflows_is_not_judged_away(U, oracle, B, Hq, Hkv, D, shape):
    """Queries so small that their norms' squares vanish, one far key so large that its norm's square is infinite: the
    score between them is the row's largest by far."""
    assert launch_shape(B, Hq, Hkv, 24, D=D)[0] == shape
    cfg = W.small_config(name="huge", kind="prefill", dtype=W.BF16, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D,
                         block_size=16, num_blocks=B * 45, ctx_lo=705, ctx_hi=705, q_len=24, seed=4)
    case = W.make_case(cfg, slopes=np.full(Hq, 0.25, np.float32))
    u = np.full(D, D ** -0.5, np.float32)
    case.q[:] = W.to_bits(u * np.float32(2.0 ** -70), W.BF16)
    case.k_cache[case.block_tables[0, 6], :, 4] = W.to_bits(u * np.float32(2.0 ** 100), W.BF16)
    widen(case)
    dev = U.DevCase(case)
    step = dev.prefill_step()
    kc, vc = oracle_filled(oracle, case)
    rows = slice(None, case.cu_q_lens[2])
    ref = oracle.paged_prefill(case.q[rows], kc, vc, case.block_tables[:2], case.context_lens[:2], case.cu_q_lens[:3],
                               case.slopes, case.scale, W.BF16)
    U.check_scaled(step[rows], ref, W.BF16, "huge")


# (sequences, heads, KV heads, head_dim): 1 and odd numbers of them, a lane's worth, one more (the plain order) - the order by length is that of one
# group of four or of eight waves, of these the latter over 8-bit caches only
@pytest.mark.parametrize("B,Hq,Hkv,D,shape,shape8", [
    (1, 8, 2, 128, "two", "two"), (3, 6, 2, 64, "two", "two"), (7, 40, 8, 128, "4", "4"), (17, 16, 16, 128, "4", "4"), (60, 16, 16, 64, "4", "8"),
    (64, 8, 2, 128, "4", "4"), (65, 8, 2, 64, "4", "4"), (64, 16, 4, 64, "4", "8"), (65, 16, 4, 128, "4", "8"), (64, 16, 4, 128, "4", "8")])
@pytest.mark.parametrize("kv8", [False, True])
def test_ragged_launches_in_order_of_length(U, oracle, kv8, B, Hq, Hkv, D, shape, shape8):
    """No slopes; chunks of up to 90 new tokens (one of up to 180) behind 0 to 200 cached ones, one sequence without any."""
    import torch
    import oracle as O
    import paper_2505_02351_amd as G
    lens = np.random.default_rng(77 + B).integers(1, 201, B).astype(np.int32)
    if B > 2:
        lens[2] = 200
    cfg = W.small_config(name="ragged", kind="prefill", dtype=W.BF16, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D,
                         block_size=16, num_blocks=B * 13 + 5, ctx_lo=1, ctx_hi=200, q_len=90, seed=77 + B)
    case = W.make_case(cfg, context_lens=lens)
    cu = case.cu_q_lens.copy()
    if B > 2:
        cu[2] = cu[1]                           # sequence 1 without new tokens, its rows sequence 2's: more of them
        assert np.diff(cu)[1] == 0 and 90 < np.diff(cu)[2] <= 180 <= lens[2]
    most = int(np.diff(cu).max())
    got, tiles = launch_shape(B, Hq, Hkv, most, D=D, slopes=False, kv8=kv8, longest=208)
    assert got == (shape8 if kv8 else shape) and (tiles > 1 or B == 1 or Hq == Hkv)
    dev = U.DevCase(case)
    dev.out.fill_(float("nan"))
    args = dev.block_tables, dev.context_lens, torch.from_numpy(cu).cuda(), None, float(case.scale)
    if kv8:
        kc, vc, dk, dv = fp8_caches(U, case, 0.0125, 0.02)
        ref = O.paged_prefill_e4m3(case.q, kc, vc, case.block_tables, case.context_lens, cu, None, case.scale, 0.0125, 0.02, W.BF16)
        G.paged_prefill_fp8(dev.out, dev.q, dk, dv, *args, 0.0125, 0.02, most)
    else:
        kc, vc = oracle_filled(oracle, case)
        ref = oracle.paged_prefill(case.q, kc, vc, case.block_tables, case.context_lens, cu, None, case.scale, W.BF16)
        dev.write_cache()
        G.paged_prefill(dev.out, dev.q, dev.k_cache, dev.v_cache, *args, most)
    torch.cuda.synchronize()
    dev.check_canaries()
    U.check_scaled(U.to_host(dev.out), ref, W.BF16, f"ragged {B}")


@pytest.mark.parametrize("distance", [2000, 8000])
def test_one_loud_far_key_does_not_cost_a_look_every_few_tiles(U, distance):
    """Chunks of 512 behind 32 000 cached tokens, slopes 2^(-8h/32): with one key of ten times the norm in every sequence the
    step takes 1.02 (1.01) of its time without, and took 3.5 (9.7) when every look read the context up to that key and
    beyond, and the next one came eight tiles later."""
    import torch
    import paper_2505_02351_amd as G
    from test_gpu_decode_unsplit_step import microseconds
    B, Hq, Hkv, D, bs, ctx, new = 4, 32, 8, 128, 16, 32000, 512
    blocks = (ctx + new) // bs
    gen = torch.Generator("cuda").manual_seed(8)
    q, k, v = (torch.randn(B * new, h, D, generator=gen, device="cuda", dtype=torch.bfloat16) for h in (Hq, Hkv, Hkv))
    kc, vc = (torch.randn(B * blocks, Hkv, bs, D, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    table = torch.randperm(B * blocks, generator=gen, device="cuda").to(torch.int32).view(B, blocks)
    lens = torch.full((B,), ctx + new, dtype=torch.int32, device="cuda")
    cu = torch.arange(0, B * new + 1, new, dtype=torch.int32, device="cuda")
    slopes = torch.exp2(-8.0 * torch.arange(1, Hq + 1, device="cuda") / Hq)
    out = torch.empty_like(q)

    def us():
        return microseconds(lambda: G.prefill_step(out, q, k, v, kc, vc, table, lens, cu, slopes, D ** -0.5, new))
    quiet = us()
    at = ctx + new - distance
    kc[table[:, at // bs].long(), :, at % bs] *= 10
    loud = us()
    assert loud <= 1.5 * quiet, (loud, quiet)


def test_fp16_rows_skip_their_far_tiles(U):
    """Chunks of 16 behind 2 048, 16 / 4 heads, slopes 2^(-8h/16), two key groups: fp16 (one output product a tile) takes
    0.84 of bf16's time (two), and took 1.5 of it when a row half of whose sum was zero wanted every tile."""
    import torch
    import paper_2505_02351_amd as G
    from test_gpu_decode_unsplit_step import microseconds
    B, Hq, Hkv, D, bs, ctx, new = 2, 16, 4, 64, 16, 2048, 16
    blocks = (ctx + new) // bs
    us = {}
    for dtype in (torch.float16, torch.bfloat16):
        gen = torch.Generator("cuda").manual_seed(9)
        q, k, v = (torch.randn(B * new, h, D, generator=gen, device="cuda").to(dtype) for h in (Hq, Hkv, Hkv))
        kc, vc = (torch.randn(B * blocks, Hkv, bs, D, generator=gen, device="cuda").to(dtype) for _ in range(2))
        table = torch.randperm(B * blocks, generator=gen, device="cuda").to(torch.int32).view(B, blocks)
        lens = torch.full((B,), ctx + new, dtype=torch.int32, device="cuda")
        cu = torch.arange(0, B * new + 1, new, dtype=torch.int32, device="cuda")
        slopes = torch.exp2(-8.0 * torch.arange(1, Hq + 1, device="cuda") / Hq)
        out = torch.empty_like(q)
        us[dtype] = microseconds(lambda: G.prefill_step(out, q, k, v, kc, vc, table, lens, cu, slopes, D ** -0.5, new))
    assert us[torch.float16] <= 1.2 * us[torch.bfloat16], us


@pytest.mark.parametrize("B,Hq,Hkv,D,new,ctx", [(2, 32, 8, 128, 40, 0), (2, 32, 8, 128, 100, 100), (2, 32, 8, 64, 40, 0),
                                                (5, 16, 4, 64, 512, 0), (8, 16, 4, 64, 160, 0)])
def test_kernels_without_a_window_are_no_slower(U, B, Hq, Hkv, D, new, ctx):
    """Without slopes, against the windowed kernel under a window that hides nothing.  Walks of 2, 7 and 2 tiles in a
    launch of few workgroups (the windowed kernel always runs one group of four waves): 0.97-1.00 of its time; 1.29, 1.12
    and 1.20 when two key groups shared such walks.  16 and 5 tiles: 1.03 and 0.97; 1.10 and 1.14 when the kernel held
    the code that looks at the rest of a walk.  GPU time: 20 calls in a graph."""
    import torch
    import paper_2505_02351_amd as G
    from test_gpu_decode_unsplit_step import microseconds
    bs = 16
    blocks = -(-(ctx + new) // bs)
    q = torch.randn(B * new, Hq, D, device="cuda", dtype=torch.bfloat16)
    kc, vc = (torch.randn(B * blocks, Hkv, bs, D, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    table = torch.arange(B * blocks, dtype=torch.int32, device="cuda").view(B, blocks)
    lens = torch.full((B,), ctx + new, dtype=torch.int32, device="cuda")
    cu = torch.arange(0, B * new + 1, new, dtype=torch.int32, device="cuda")
    out = torch.empty_like(q)

    def us(call):
        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                call()
        return microseconds(graph.replay, reps=1, runs=15) / 20
    plain = us(lambda: G.paged_prefill(out, q, kc, vc, table, lens, cu, None, D ** -0.5, new))
    windowed = us(lambda: G.paged_prefill_window(out, q, kc, vc, table, lens, cu, None, D ** -0.5, 4096, new))
    assert plain <= 1.08 * windowed, (plain, windowed)
