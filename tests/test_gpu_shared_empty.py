"""Shared prefixes, bundles with an empty slot whose shared_blocks entry and query row were left behind: a column of nobody's,
which must not touch the others' arithmetic (a live column moves the references of its whole wave's)."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import U  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [12, 64, 68])         # up to 64 sequences a segment's extent comes from lanes, beyond from memory
@pytest.mark.parametrize("dtype,D", [(W.BF16, 128), (W.F16, 64)])
@pytest.mark.parametrize("fused", [True, False])
def test_an_empty_members_left_over_entry_changes_nothing(U, fused, dtype, D, B):
    import torch
    Hq, Hkv, bs, blocks = 16, 4, 16, 20             # bundles of four
    ctx = blocks * bs + 40
    cfg = W.small_config(name="empty member", dtype=dtype, batch=B, num_heads=Hq, num_kv_heads=Hkv, head_dim=D, block_size=bs,
                         num_blocks=B * -(-ctx // bs) + 3, ctx_lo=ctx, ctx_hi=ctx, seed=5 + B)
    case = W.make_case(cfg)
    for b in range(B):
        case.block_tables[b, :blocks] = case.block_tables[b - b % 4, :blocks]
    shared = np.array([blocks if b % 4 else 0 for b in range(B)], np.int32)
    empty = np.arange(B) % 4 == 2                   # (leader and two members are live)
    case.slopes = None
    case.q[empty] = W.to_bits(64.0 * W.from_bits(case.q[empty], dtype).astype(np.float32), dtype)
    dev = U.DevCase(case)
    lens = case.context_lens.copy()
    lens[empty] = 0
    dev.context_lens = torch.from_numpy(lens).to("cuda")
    got = dev.decode_shared(shared, fused=fused)
    want = dev.decode_shared(np.where(empty, 0, shared).astype(np.int32), fused=fused)
    assert not got[empty].any()
    assert (got == want).all()
