"""The tail expansions with long tails: the workgroup shapes that the launch chooses by the number of stages and tiles, up to tens
of thousands of tiles.  Each against the one-shot expansion of the same positions, bit for bit; positions
ahead of the tail stay untouched."""
import pytest
import torch

pytestmark = pytest.mark.gpu

R_KV, D_R = 512, 64


@pytest.mark.parametrize("nb,tail,page,g,d_h,d_v,fp8", [
    (70, 64, 64, 1, 128, 128, False),       # 140 tiles x 8 halves: two waves per workgroup
    (70, 64, 64, 1, 128, 128, True),
    (33, 31, 64, 1, 128, 128, False),       # 32 tiles, the last of 31 tokens: one wave
    (65, 63, 64, 1, 128, 128, False),       # 128 tiles, the last of 31 tokens: two waves
    (70, 64, 64, 2, 128, 128, False),       # more than four stages: one wave however many
    (70, 64, 64, 1, 192, 256, False),
    (2100, 1024, 1024, 1, 128, 128, False),  # 67 200 tiles
    (2100, 1024, 1024, 2, 128, 128, False),
])
def test_long_tail_equals_one_shot(nb, tail, page, g, d_h, d_v, fp8):
    from paper_2605_15250_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(11)
    max_pages = 3 if page == 64 else 1
    held = [b for b in range(nb) if page == 64 or b in (0, 1, 777, nb - 2, nb - 1)]   # sequences whose pages are in the pool
    num_pages = len(held) * max_pages
    table = torch.full((nb, max_pages), -1, dtype=torch.int32)
    for k, b in enumerate(held):
        table[b] = torch.arange(k * max_pages, (k + 1) * max_pages, dtype=torch.int32)
    lens = [(37 * b) % (max_pages * page) + 1 for b in range(nb)]          # some shorter than the tail
    d_table, d_lens = table.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
    pool = torch.randn(num_pages, page, R_KV + D_R, generator=gen, device="cuda").bfloat16()
    w_uk = (torch.randn(g, R_KV, d_h, generator=gen, device="cuda") * R_KV ** -0.5).bfloat16()
    w_uv = (torch.randn(g, R_KV, d_v, generator=gen, device="cuda") * R_KV ** -0.5).bfloat16()
    shape = B.make_shape(nb, g, g, d_h, R_KV, D_R, 1, B.GQLA_BF16, 0.0, d_v)
    ws = torch.empty(B.gqla_expand_workspace_bytes(shape, g), dtype=torch.uint8, device="cuda")
    latent = B.make_cache(pool, d_lens, d_table, page, max_pages, num_pages)
    eb, fill = (1 if fp8 else 2), 0xA5
    outs = [torch.full((num_pages, page * (g * (d_h + d_v) * eb + D_R * 2)), fill, dtype=torch.uint8, device="cuda") for _ in range(2)]
    caches = [B.make_cache(o, d_lens, d_table, page, max_pages, num_pages, g) for o in outs]
    print("tail", nb, tail, g, d_h, flush=True)
    if fp8:
        B.gqla_expand_cache_tail_fp8(shape, latent, w_uk, w_uv, 0, g, caches[0], tail, 2.0 ** -6, 2.0 ** -6, ws)
        B.gqla_expand_cache_fp8(shape, latent, w_uk, w_uv, 0, g, caches[1], 2.0 ** -6, 2.0 ** -6, ws)
    else:
        B.gqla_expand_cache_tail(shape, latent, w_uk, w_uv, 0, g, caches[0], tail, ws)
        B.gqla_expand_cache(shape, latent, w_uk, w_uv, 0, g, caches[1], ws)
    torch.cuda.synchronize()

    def by_token(o):       # [sequence of the pool][token] -> all bytes of the token, in one order
        o = o.reshape(len(held), max_pages, -1)
        k, v = g * d_h * page * eb, g * d_v * page * eb
        if fp8:            # [g][d_h / 16][P][16] and [g][P / 32][d_h][2][16]: slot 32 T + 16 u + 8 h + i at [T][d][h][8 u + i]
            kk = o[..., :k].reshape(len(held), max_pages, g * (d_h // 16), page, 16).transpose(2, 3)
            vv = o[..., k:k + v].reshape(len(held), max_pages, g, page // 32, d_v, 2, 2, 8).permute(0, 1, 3, 6, 5, 7, 2, 4)
        else:              # [g][d_h / 8][P][8] and [g][P / 8][d_v][8] of 16-bit elements
            kk = o[..., :k].reshape(len(held), max_pages, g * (d_h // 8), page, 16).transpose(2, 3)
            vv = o[..., k:k + v].reshape(len(held), max_pages, g, page // 8, d_v, 8, 2).permute(0, 1, 3, 5, 2, 4, 6)
        rr = o[..., k + v:].reshape(len(held), max_pages, D_R // 8, page, 16).transpose(2, 3)
        return torch.cat([x.reshape(len(held), max_pages * page, -1) for x in (kk, vv, rr)], 2)
    got, want = by_token(outs[0]), by_token(outs[1])
    pos = torch.arange(max_pages * page, device="cuda")
    n = torch.tensor([lens[b] for b in held], device="cuda")[:, None]
    in_tail = (pos >= n - tail) & (pos < n)
    assert torch.equal(got[in_tail], want[in_tail])
    assert bool((got[~in_tail] == fill).all())
