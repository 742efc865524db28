"""Single-pass decode calls with many output rows write them past the dies' L2s and in windows of the clock; neither may change a bit.

A batch large enough for that is compared with the same sequences in two calls that are not (GPU only); the launches' arithmetic is that of
the calls the oracle checks elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PAGE = 16


@pytest.mark.parametrize("kv,d,Hq,Hkv,B,longest,append", [
    ("bf16", 128, 64, 8, 340, 900, True),      # 11 MB of rows, windows; the newest token comes as a row
    ("bf16", 128, 28, 4, 740, 512, False),     # written through, no windows (256 KB of K/V per head at most)
    ("bf16", 64, 40, 8, 1040, 1600, False),
    ("bf16", 128, 40, 2, 520, 800, False),     # 20 query heads per KV head: two blocks of rows, 16 and 4
    ("fp8", 128, 64, 8, 340, 2000, False),
    ("fp8", 64, 48, 16, 860, 700, False),
    ("fp8", 64, 64, 2, 660, 3300, False),      # windows at head_dim 64; 32 query heads per KV head
])
def test_many_rows_equal_the_same_rows_of_smaller_calls(kv, d, Hq, Hkv, B, longest, append):
    import torch

    import paper_2508_11553_amd as sd

    gen = torch.Generator(device="cuda").manual_seed(B)
    rng = np.random.default_rng(B)
    lens = rng.integers(0, longest + 1, B)
    lens[:3] = [1, longest, 0]
    nb = (lens + PAGE - 1) // PAGE
    table = np.zeros((B, -(-longest // PAGE)), np.int32)
    place = rng.permutation(int(nb.sum()))
    for b, end in enumerate(np.cumsum(nb)):
        table[b, :nb[b]] = place[end - nb[b]:end]
    pages = max(1, len(place))
    if kv == "bf16":
        k, v = (torch.randn((pages, Hkv, PAGE, d), generator=gen, device="cuda").bfloat16().view(torch.int16) for _ in range(2))
        ks = vs = None
    else:
        k, v = (torch.randint(0, 0x77, (pages, Hkv, PAGE, d), generator=gen, device="cuda", dtype=torch.uint8) for _ in range(2))
        ks, vs = (torch.rand((pages, Hkv), generator=gen, device="cuda") * 0.01 + 0.001 for _ in range(2))
    q, k_new, v_new = (torch.randn((B, h, d), generator=gen, device="cuda").bfloat16().view(torch.int16) for h in (Hq, Hkv, Hkv))
    table, lens = torch.tensor(table, device="cuda"), torch.tensor(lens.astype(np.int32), device="cuda")

    def call(first, end):
        shape = sd.Shape(batch=end - first, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=PAGE, num_pages=pages,
                         max_blocks_per_seq=table.shape[1], kv_dtype=sd.SD_BF16 if kv == "bf16" else sd.SD_FP8_E4M3,
                         max_context_len=longest, chunk_tokens=-(-longest // 128) * 128)
        out = torch.full((end - first, Hq, d), float("nan"), device="cuda")
        n = sd.workspace_bytes(shape)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        pools = [k.clone(), v.clone()] if append else [k, v]
        row = slice(first, end)
        if append:
            sd.paged_decode_attention_append(shape, q[row].clone(), k_new[row].clone(), v_new[row].clone(), *pools,
                                             table[row].clone(), lens[row].clone(), 0.1, out, ws, n)
        else:
            sd.paged_decode_attention(shape, q[row].clone(), *pools, ks, vs, table[row].clone(), lens[row].clone(), 0.1, out, ws, n)
        torch.cuda.synchronize()
        return out, pools

    whole, pools = call(0, B)
    assert whole.numel() * 4 >= 10 << 20 and not torch.isnan(whole).any()
    cut = B // 2 & ~1
    parts = [call(0, cut), call(cut, B)]
    assert all(p[0].numel() * 4 < 10 << 20 for p in parts)
    assert torch.equal(whole, torch.cat([p[0] for p in parts]))
    if append:   # every sequence's newest row went into the pool
        for pool, new in zip(pools, (k_new, v_new)):
            at = (lens.long() - 1).clamp(min=0)
            got = pool[table[torch.arange(B, device="cuda"), at // PAGE].long(), :, at % PAGE]
            assert torch.equal(got[lens > 0], new[lens > 0])
