"""Page-table rows far wider than any sequence: what a row could hold (max_pages * page_size tokens) may pass 2^31 and bounds the
launch of the cache switches; the results are those of a row that just holds the sequences, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu

P, R_KV, D_R, D, G = 1024, 512, 64, 128, 4
LENS = [300, 1100]


def _switch(op, nb, max_pages):
    from paper_2605_15250_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(3)
    num_pages, lens = 3, LENS[:nb]
    need = [-(-n // P) for n in lens]
    table, at = torch.full((nb, max_pages), -1, dtype=torch.int32), 0
    for b, n in enumerate(need):
        table[b, :n] = torch.arange(at, at + n, dtype=torch.int32)
        at += n
    d_table, d_lens = table.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
    f32 = op == "expand_f32"
    shape = B.make_shape(nb, G, G, D, R_KV, D_R, 1, B.GQLA_F32 if f32 else B.GQLA_BF16)

    def values(*size):
        return torch.randn(*size, generator=gen, device="cuda").to(torch.float32 if f32 else torch.bfloat16)

    def cache(pool, groups=0):
        return B.make_cache(pool, d_lens, d_table, P, max_pages, num_pages, groups)
    latent, keys = values(num_pages, P * (R_KV + D_R)), values(num_pages, P * (2 * G * D + D_R))
    w_uk, w_uv, w_inv = values(G, R_KV, D), values(G, R_KV, D), values(R_KV, G * D)
    ws = torch.empty(max(16, B.gqla_expand_workspace_bytes(shape, G)), dtype=torch.uint8, device="cuda")
    print(op, nb, max_pages, flush=True)
    if op in ("expand", "expand_f32"):
        out = torch.zeros_like(keys)
        B.gqla_expand_cache(shape, cache(latent), w_uk, w_uv, 0, G, cache(out, G), ws)
    elif op == "expand_fp8":
        out = torch.zeros(num_pages, P * B.gqla_expanded_fp8_bytes_per_token(G, D, D_R), dtype=torch.uint8, device="cuda")
        B.gqla_expand_cache_fp8(shape, cache(latent), w_uk, w_uv, 0, G, cache(out, G), 1.0, 1.0, ws)
    else:
        out = torch.zeros_like(latent)
        B.gqla_compress_cache(shape, cache(keys, G), w_inv, cache(out))
    torch.cuda.synchronize()
    return out


# (a grid over what two such rows hold, or one of the compression, would not fit a launch)
@pytest.mark.parametrize("op,nb", [("expand", 1), ("expand_fp8", 1), ("expand", 2), ("expand_fp8", 2), ("compress", 1), ("compress", 2), ("expand_f32", 1)])
def test_row_of_two_to_the_31_tokens(op, nb):
    narrow = _switch(op, nb, 2)
    assert int((narrow != 0).sum()) > 0
    assert torch.equal(_switch(op, nb, 1 << 21), narrow)


@pytest.mark.parametrize("op,d_h,d_v", [("expand", 128, 128), ("expand", 192, 256), ("compress", 128, 128), ("compress", 192, 256)])
def test_more_blocks_than_workgroups(op, d_h, d_v):
    """Beyond 2048 workgroups one takes several blocks in turn: sequences whose pages are a few shared ones, so that every
    sequence's result has to be that of the first with its length (the same bits for the expansion; the compression starts its
    sums at another place from tile to tile, which moves them by the order of fp32 sums)."""
    from paper_2605_15250_amd import binding as B
    g, page = 4, 64
    block = 256 if op == "expand" else 128
    gen = torch.Generator(device="cuda").manual_seed(4)
    lens = [3 * block, 2 * block + 70, 1, 0, block] * (2100 // 8)      # eight blocks in five sequences: 2096 and a few more
    lens += [3 * block] * 2 + [5]
    nb, per = len(lens), 3 * block // page
    n_out = nb * per
    wide_in = torch.randn(per, page * ((R_KV + D_R) if op == "expand" else g * (d_h + d_v) + D_R), generator=gen, device="cuda").bfloat16()
    t_in = torch.arange(per, dtype=torch.int32).repeat(nb, 1).cuda()
    d_lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    shape = B.make_shape(nb, g, g, d_h, R_KV, D_R, 1, B.GQLA_BF16, 0.0, d_v)
    out = torch.zeros(n_out, page * ((R_KV + D_R) if op != "expand" else g * (d_h + d_v) + D_R), dtype=torch.bfloat16, device="cuda")
    src = B.make_cache(wide_in, d_lens, t_in, page, per, per, 0 if op == "expand" else g)
    dst = B.make_cache(out, d_lens, None, page, per, n_out, g if op == "expand" else 0)
    print(op, d_h, nb, flush=True)
    if op == "expand":
        w_uk = (torch.randn(g, R_KV, d_h, generator=gen, device="cuda") * R_KV ** -0.5).bfloat16()
        w_uv = (torch.randn(g, R_KV, d_v, generator=gen, device="cuda") * R_KV ** -0.5).bfloat16()
        ws = torch.empty(B.gqla_expand_workspace_bytes(shape, g), dtype=torch.uint8, device="cuda")
        B.gqla_expand_cache(shape, src, w_uk, w_uv, 0, g, dst, ws)
    else:
        w_inv = (torch.randn(R_KV, g * d_h, generator=gen, device="cuda") * (g * d_h) ** -0.5).bfloat16()
        B.gqla_compress_cache(shape, src, w_inv, dst)
    torch.cuda.synchronize()
    seqs = out.reshape(nb, per, -1)
    for n in sorted(set(lens)):
        same = seqs[[b for b in range(nb) if lens[b] == n]].float()
        assert bool(torch.isfinite(same).all()) and (n == 0) == (int((same != 0).sum()) == 0)
        # fp32 sums of up to 768 products in another order, then one rounding to bf16: a step of 2^-8 of the value at most
        bound = 0.0 if op == "expand" else same[:1].abs() * 2.0 ** -7 + 1e-4
        assert bool(((same - same[:1]).abs() <= bound).all()), n
