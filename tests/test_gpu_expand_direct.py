"""The ways the expansion shares its work out, each against another of them, bit for bit: weights as the caller holds them (few
blocks, few tail tokens) against repacked ones, at the edges between the two -- 72 blocks that the page-table rows could hold,
256 tail tokens -- and on ragged, padded and empty rows, slices of the groups and both pairs of dims; a last round whose
(block, group) pairs are dealt out evenly."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _setup(g, d_h, d_v, lens, max_pages, seed=5):
    from paper_2605_15250_amd import binding as B
    P, r_kv, d_r = 64, 512, 64
    gen = torch.Generator(device="cuda").manual_seed(seed)
    nb = len(lens)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").bfloat16()
    need = max(-(-n // P) for n in lens)
    num_pages = nb * need
    table = np.full((nb, max_pages), -1, np.int32)
    table[:, :need] = np.random.default_rng(seed).permutation(num_pages).reshape(nb, need)
    return B, dict(P=P, r_kv=r_kv, d_r=d_r, nb=nb, num_pages=num_pages, max_pages=max_pages, table=torch.from_numpy(table).cuda(),
                   lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), pool=rnd(num_pages, P, r_kv + d_r),
                   w_uk=rnd(g, r_kv, d_h) * r_kv ** -0.5, w_uv=rnd(g, r_kv, d_v) * r_kv ** -0.5)


def _cache(B, s, pool, width, groups=0):
    """A view of the same pages with page-table rows of `width` entries."""
    table = s["table"][:, :width].contiguous()
    return B.make_cache(pool, s["lens"], table, s["P"], width, s["num_pages"], groups), table


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("g,first,count,d_h,d_v,lens", [
    (8, 0, 8, 128, 128, [1, 63, 64, 65, 255, 256, 257, 300]),
    (4, 1, 2, 128, 128, [700, 0, 31]),                   # a slice of two groups
    (5, 0, 5, 192, 256, [513, 90]),                      # seven stages a group
    (1, 0, 1, 128, 128, [256 * 9 + 5]),                  # one group: nothing to share out
    (32, 1, 24, 128, 128, [70] * 64),                    # 24 groups in four shares: six a workgroup
    (32, 1, 25, 128, 128, [70] * 64),                    # seven: repacked
])
def test_one_shot(g, first, count, d_h, d_v, lens, fp8):
    if fp8 and d_h != 128:
        pytest.skip("the 8-bit expanded cache has key and value dims of 128")
    need = max(-(-n // 64) for n in lens)
    wide = max(need, 4 * 73)                             # rows that could hold more than 72 blocks: repacked weights
    B, s = _setup(g, d_h, d_v, lens, wide)
    shape = B.make_shape(s["nb"], 4 * g, g, d_h, s["r_kv"], s["d_r"], 1, B.GQLA_BF16, 0.0, d_v)
    ws = torch.empty(B.gqla_expand_workspace_bytes(shape, count), dtype=torch.uint8, device="cuda")
    elems = B.gqla_expanded_fp8_bytes_per_token(count, d_h, s["d_r"]) if fp8 else 2 * (count * (d_h + d_v) + s["d_r"])
    got = []
    for width in (need, wide):
        out = torch.full((s["num_pages"] * 64 * elems,), 0x5A, dtype=torch.uint8, device="cuda")
        lat, t1 = _cache(B, s, s["pool"], width)
        exp, t2 = _cache(B, s, out, width, count)
        print("expand direct", g, first, count, d_h, fp8, width, flush=True)
        if fp8:
            B.gqla_expand_cache_fp8(shape, lat, s["w_uk"], s["w_uv"], first, count, exp, 0.02, 0.03, ws)
        else:
            B.gqla_expand_cache(shape, lat, s["w_uk"], s["w_uv"], first, count, exp, ws)
        torch.cuda.synchronize()
        got.append(out)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("g,count,d_h,d_v,lens,wide,repacked", [
    (8, 8, 128, 128, [300, 70], False, False),
    (8, 8, 128, 128, [300, 70], True, True),             # the page-table rows could hold more than 72 blocks
    (32, 24, 128, 128, [70] * 64, False, False),         # 24 groups in four shares: six a workgroup
    (32, 25, 128, 128, [70] * 64, False, True),          # seven
    (1, 1, 192, 256, [200], False, True),                # (192, 256)
    (8, 8, 192, 256, [20, 250], False, True),
])
def test_one_shot_form(g, count, d_h, d_v, lens, wide, repacked):
    """Which calls repack the weights: those whose last waves, of fewer than 64 tokens, would lose more than the launch costs.  The
    scratch shows it."""
    need = max(-(-n // 64) for n in lens)
    width = 4 * 73 if wide else need
    B, s = _setup(g, d_h, d_v, lens, width)
    shape = B.make_shape(s["nb"], g, g, d_h, s["r_kv"], s["d_r"], 1, B.GQLA_BF16, 0.0, d_v)
    ws = torch.full((B.gqla_expand_workspace_bytes(shape, count),), 0x5A, dtype=torch.uint8, device="cuda")
    out = torch.zeros(s["num_pages"] * 64 * (count * (d_h + d_v) + s["d_r"]), dtype=torch.bfloat16, device="cuda")
    lat, t1 = _cache(B, s, s["pool"], width)
    exp, t2 = _cache(B, s, out, width, count)
    print("expand form", g, count, d_h, wide, flush=True)
    B.gqla_expand_cache(shape, lat, s["w_uk"], s["w_uv"], 0, count, exp, ws)
    torch.cuda.synchronize()
    assert bool((ws != 0x5A).any()) == repacked


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("g,d_h,d_v,nb,tail", [
    (8, 128, 128, 1, 1),
    (8, 128, 128, 33, 2),                                # 66 tokens: the third tile holds two
    (1, 128, 128, 128, 2),                               # 256 tokens, the last without the repacking
    (1, 128, 128, 129, 2),                               # 258: repacked
    (5, 192, 256, 7, 3),
])
def test_tail(g, d_h, d_v, nb, tail, fp8):
    if fp8 and d_h != 128:
        pytest.skip("the 8-bit expanded cache has key and value dims of 128")
    lens = [tail + (37 * i) % 150 for i in range(nb)]
    if nb > 1:
        lens[-1] = tail - 1                              # shorter than the tail: its first position does not exist
    B, s = _setup(g, d_h, d_v, lens, max(-(-n // 64) for n in lens))
    shape = B.make_shape(nb, 4 * g, g, d_h, s["r_kv"], s["d_r"], 1, B.GQLA_BF16, 0.0, d_v)
    ws = torch.empty(B.gqla_expand_workspace_bytes(shape, g), dtype=torch.uint8, device="cuda")
    elems = B.gqla_expanded_fp8_bytes_per_token(g, d_h, s["d_r"]) if fp8 else 2 * (g * (d_h + d_v) + s["d_r"])
    lat, t1 = _cache(B, s, s["pool"], s["max_pages"])
    outs = [torch.full((s["num_pages"] * 64 * elems,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(2)]
    caches = [_cache(B, s, o, s["max_pages"], g) for o in outs]
    print("tail direct", g, d_h, nb, tail, fp8, flush=True)
    if fp8:       # one call for all tokens of the whole context gives the codes of every position
        B.gqla_expand_cache_tail_fp8(shape, lat, s["w_uk"], s["w_uv"], 0, g, caches[0][0], tail, 0.02, 0.03, ws)
        B.gqla_expand_cache_fp8(shape, lat, s["w_uk"], s["w_uv"], 0, g, caches[1][0], 0.02, 0.03, ws)
    else:
        B.gqla_expand_cache_tail(shape, lat, s["w_uk"], s["w_uv"], 0, g, caches[0][0], tail, ws)
        B.gqla_pack_expand_weights(shape, s["w_uk"], s["w_uv"], 0, g, ws)
        B.gqla_expand_cache_tail_packed(shape, lat, ws, g, caches[1][0], tail)
    torch.cuda.synchronize()
    if not fp8:
        assert torch.equal(outs[0], outs[1])
    else:         # bytes that the tail wrote are those of the whole expansion; the others were not touched
        wrote = outs[0] != 0x5A
        assert torch.equal(outs[0][wrote], outs[1][wrote])
        assert int(wrote.sum()) >= sum(min(n, tail) for n in lens) * elems * 0.9     # (a code may equal the fill)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("g,d_h,d_v,tokens,repacked", [
    (48, 128, 128, 256, False),                          # 192 stages, eight tiles
    (64, 128, 128, 192, False),                          # 256, six
    (64, 128, 128, 193, True),                           # seven
    (80, 128, 128, 96, False),                           # 320, three
    (65, 128, 128, 97, True),                            # 260, four
    (96, 128, 128, 65, True),                            # 384, three
    (128, 128, 128, 32, False),                          # 512, one
    (128, 128, 128, 33, True),                           # two
    (64, 192, 256, 32, False),                           # 448, one
    (64, 192, 256, 64, True),                            # two
])
def test_tail_of_many_groups(g, d_h, d_v, tokens, repacked, fp8):
    """Weights far beyond the caches are repacked from fewer tokens on (each tile of 32 tokens reads them all); the scratch shows
    which form ran.  Against the whole expansion: the same bits."""
    if fp8 and d_h != 128:
        pytest.skip("the 8-bit expanded cache has key and value dims of 128")
    lens = [1 + (37 * i) % 90 for i in range(tokens)]
    B, s = _setup(g, d_h, d_v, lens, max(-(-n // 64) for n in lens))
    shape = B.make_shape(tokens, g, g, d_h, s["r_kv"], s["d_r"], 1, B.GQLA_BF16, 0.0, d_v)
    elems = B.gqla_expanded_fp8_bytes_per_token(g, d_h, s["d_r"]) if fp8 else 2 * (g * (d_h + d_v) + s["d_r"])
    lat, t1 = _cache(B, s, s["pool"], s["max_pages"])
    outs = [torch.full((s["num_pages"] * 64 * elems,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(2)]
    scales = (0.02, 0.03) if fp8 else ()
    print("tail many groups", g, d_h, tokens, fp8, flush=True)
    ws = torch.full((B.gqla_expand_workspace_bytes(shape, g),), 0x5A, dtype=torch.uint8, device="cuda")
    exp, t2 = _cache(B, s, outs[0], s["max_pages"], g)
    (B.gqla_expand_cache_tail_fp8 if fp8 else B.gqla_expand_cache_tail)(shape, lat, s["w_uk"], s["w_uv"], 0, g, exp, 1, *scales, ws)
    torch.cuda.synchronize()
    assert bool((ws != 0x5A).any()) == repacked
    exp, t2 = _cache(B, s, outs[1], s["max_pages"], g)
    (B.gqla_expand_cache_fp8 if fp8 else B.gqla_expand_cache)(shape, lat, s["w_uk"], s["w_uv"], 0, g, exp, *scales, ws)
    torch.cuda.synchronize()
    wrote = outs[0] != 0x5A
    assert torch.equal(outs[0][wrote], outs[1][wrote])
    assert int(wrote.sum()) >= tokens * elems * 0.9      # (a byte may equal the fill)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("g,d_h,d_v,blocks", [
    (8, 128, 128, 129),                                  # the fewest whose (block, group) pairs are dealt out evenly
    (8, 128, 128, 192),                                  # the most: six groups a workgroup
    (8, 128, 128, 193),                                  # one block a workgroup
    (8, 128, 128, 256 + 150),                            # behind a whole round
    (3, 128, 128, 82),                                   # shares of one and two groups, as before
    (5, 192, 256, 150),
])
def test_last_round_dealt_out_evenly(g, d_h, d_v, blocks, fp8):
    """One call over all sequences against calls over 40 of them at a time: the same bits."""
    if fp8 and d_h != 128:
        pytest.skip("the 8-bit expanded cache has key and value dims of 128")
    lens = [1 + (29 * i) % 90 for i in range(blocks - 2)] + [300]
    B, s = _setup(g, d_h, d_v, lens, 292)                # rows that could hold 73 blocks: repacked weights in every call
    ws = torch.empty(g * s["r_kv"] * (d_h + d_v) * 2, dtype=torch.uint8, device="cuda")
    elems = B.gqla_expanded_fp8_bytes_per_token(g, d_h, s["d_r"]) if fp8 else 2 * (g * (d_h + d_v) + s["d_r"])
    outs = []
    for step in (len(lens), 40):
        out = torch.full((s["num_pages"] * 64 * elems,), 0x5A, dtype=torch.uint8, device="cuda")
        for b0 in range(0, len(lens), step):
            lens_d, table = s["lens"][b0:b0 + step].clone(), s["table"][b0:b0 + step].contiguous()
            shape = B.make_shape(len(lens_d), 4 * g, g, d_h, s["r_kv"], s["d_r"], 1, B.GQLA_BF16, 0.0, d_v)
            lat = B.make_cache(s["pool"], lens_d, table, 64, 292, s["num_pages"])
            exp = B.make_cache(out, lens_d, table, 64, 292, s["num_pages"], g)
            print("expand even", g, d_h, blocks, fp8, step, b0, flush=True)
            if fp8:
                B.gqla_expand_cache_fp8(shape, lat, s["w_uk"], s["w_uv"], 0, g, exp, 0.02, 0.03, ws)
            else:
                B.gqla_expand_cache(shape, lat, s["w_uk"], s["w_uv"], 0, g, exp, ws)
            torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
