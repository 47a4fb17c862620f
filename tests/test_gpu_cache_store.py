"""GPU parity of the cache stores at token rows that are not a power of two of pieces, at row strides and alignments that
take either width of access, with padding tokens: bit copies and E4M3 codes, compared with torch's indexing and conversion."""
import pytest

from test_gpu_parity import U  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,D,bs", [(1, 64, 16), (3, 128, 16), (5, 64, 32), (7, 128, 64), (8, 128, 16), (9, 64, 16)])
@pytest.mark.parametrize("tokens", [1, 2, 85, 1027])
@pytest.mark.parametrize("kind", ["rows", "strided", "odd", "e4m3", "e4m3 heads"])
def test_new_rows_lie_where_their_slots_say(U, kind, tokens, Hkv, D, bs):
    import torch
    import paper_2505_02351_amd as G
    gen = torch.Generator().manual_seed(1000 * Hkv + tokens)
    blocks = -(-tokens // bs) + 3
    slots = torch.randperm(blocks * bs, generator=gen)[:tokens]
    slots[::11] = -1                                            # padding: nothing is stored
    pad = {"rows": 0, "odd": 1}.get(kind, 8)                    # elements from one token's row to the next beyond the row

    def rows():
        flat = torch.randn(tokens * (Hkv * D + pad) + 8, generator=gen).to(torch.bfloat16).cuda()
        return flat[8 if pad != 1 else 1:][:tokens * (Hkv * D + pad)].view(tokens, Hkv * D + pad)[:, :Hkv * D].view(tokens, Hkv, D)
    k, v = rows(), rows()
    e4m3 = kind.startswith("e4m3")
    caches = [torch.randint(0, 120, (blocks, Hkv, bs, D), generator=gen, dtype=torch.uint8).cuda() for _ in range(2)]
    if not e4m3:
        caches = [c.to(torch.bfloat16) for c in caches]
    want = [c.clone() for c in caches]
    scales = torch.tensor([[0.01 + 0.001 * g for g in range(Hkv)], [0.02 - 0.001 * g for g in range(Hkv)]]).cuda()
    kept = slots >= 0
    at = slots[kept].cuda()
    for i, (c, x) in enumerate(zip(want, (k, v))):
        x = x[kept.cuda()]
        if e4m3:
            inv = 1.0 / (scales[i] if kind == "e4m3 heads" else scales[i, :1].expand(Hkv))
            x = (x.float() * inv[None, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
        c[at // bs, :, at % bs] = x
    if kind == "e4m3":
        G.reshape_and_cache_fp8(k, v, *caches, slots.cuda(), float(scales[0, 0]), float(scales[1, 0]))
    elif kind == "e4m3 heads":
        G.reshape_and_cache_fp8_heads(k, v, *caches, slots.cuda(), scales[0], scales[1])
    else:
        G.reshape_and_cache(k, v, *caches, slots.cuda())
    torch.cuda.synchronize()
    for got, ref, name in zip(caches, want, "kv"):
        assert torch.equal(got.view(torch.uint8), ref.view(torch.uint8)), name
