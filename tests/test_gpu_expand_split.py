"""gqla_expand_cache with the groups shared out over workgroups: the kernel does so when the blocks of 256 tokens that the
lengths make leave compute units idle (256 // blocks shares, at most one per group, none smaller than needed).  Each case is
compared bit for bit with expanding the groups one by one, and with the fp64 product; empty and short sequences sit between
longer ones."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _lens(blocks):
    """Sequences of 0 to 300 tokens that make `blocks` blocks."""
    lens = []
    for n in [300, 0, 129, 256, 1, 257, 200] * blocks:
        n_blocks = -(-n // 256)
        if n_blocks > blocks:
            continue
        lens.append(n)
        blocks -= n_blocks
        if blocks == 0:
            return lens


def _shares(blocks, g):
    """Groups of each share, by the rule in the kernel's comment."""
    p = min(256 // blocks, g)
    per = -(-g // p)
    parts = -(-g // per)
    return [g * (k + 1) // parts - g * k // parts for k in range(parts)]


@pytest.mark.parametrize("blocks,g,d_h,d_v,fp8,shares,row_pages", [
    (5, 8, 128, 128, False, [1] * 8, 0),         # one workgroup per group
    (40, 8, 128, 128, False, [2] * 4, 0),        # shares that start behind group 0 and hold several groups
    (80, 8, 128, 128, False, [2, 3, 3], 0),      # ... of different sizes
    (80, 8, 128, 128, False, [2, 3, 3], 160),    # the same from rows wider than the sequences
    (160, 8, 128, 128, False, [8], 0),           # not shared out
    (80, 5, 192, 256, False, [1, 2, 2], 0),      # an odd number of stages per group: shares start at odd stages
    (120, 5, 192, 256, False, [2, 3], 0),
    (40, 8, 128, 128, True, [2] * 4, 0),
    (80, 8, 128, 128, True, [2, 3, 3], 0),
    (160, 8, 128, 128, True, [8], 0),
])
def test_expand_shares_equal_single_groups(blocks, g, d_h, d_v, fp8, shares, row_pages):
    from paper_2605_15250_amd import binding as B
    assert _shares(blocks, g) == shares
    r_kv, d_r, P, lens = 512, 64, 64, _lens(blocks)
    nb, need = len(lens), [-(-n // P) for n in lens]
    assert sum(-(-n // 256) for n in lens) == blocks
    num_pages, max_pages = sum(need) + 3, max(row_pages, max(need))
    gen = torch.Generator(device="cuda").manual_seed(5)
    perm = torch.randperm(num_pages, generator=gen, device="cuda").cpu().tolist()
    table = torch.full((nb, max_pages), -1, dtype=torch.int32)
    at = 0
    for b, n in enumerate(need):
        table[b, :n] = torch.tensor(perm[at:at + n], dtype=torch.int32)
        at += n
    d_table, d_lens = table.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
    pool = torch.randn(num_pages, P, r_kv + d_r, generator=gen, device="cuda").bfloat16()
    w_uk = (torch.randn(g, r_kv, d_h, generator=gen, device="cuda") * r_kv ** -0.5).bfloat16()
    w_uv = (torch.randn(g, r_kv, d_v, generator=gen, device="cuda") * r_kv ** -0.5).bfloat16()
    shape = B.make_shape(nb, g, g, d_h, r_kv, d_r, 1, B.GQLA_BF16, 0.0, d_v)
    ws = torch.empty(B.gqla_expand_workspace_bytes(shape, g), dtype=torch.uint8, device="cuda")
    latent = B.make_cache(pool, d_lens, d_table, P, max_pages, num_pages)
    eb = 1 if fp8 else 2
    fill = 0xA5

    def expand(begin, count):
        out = torch.full((num_pages, P * (count * (d_h + d_v) * eb + d_r * 2)), fill, dtype=torch.uint8, device="cuda")
        cache = B.make_cache(out, d_lens, d_table, P, max_pages, num_pages, count)
        print("expand", blocks, begin, count, flush=True)
        if fp8:
            B.gqla_expand_cache_fp8(shape, latent, w_uk, w_uv, begin, count, cache, 2.0 ** -6, 2.0 ** -6, ws)
        else:
            B.gqla_expand_cache(shape, latent, w_uk, w_uv, begin, count, cache, ws)
        torch.cuda.synchronize()
        return out
    full = expand(0, g)
    kb, vb = P * d_h * eb, P * d_v * eb
    for j in range(g):
        one = expand(j, 1)
        assert torch.equal(full[:, j * kb:(j + 1) * kb], one[:, :kb]), "keys of group %d" % j
        assert torch.equal(full[:, g * kb + j * vb:g * kb + (j + 1) * vb], one[:, kb:kb + vb]), "values of group %d" % j
        assert torch.equal(full[:, g * (kb + vb):], one[:, kb + vb:]), "k_R"
    if not fp8:
        keys = full.view(torch.bfloat16)[:, : g * P * d_h].reshape(num_pages, g, d_h // 8, P, 8).permute(0, 3, 1, 2, 4).reshape(num_pages, P, g, d_h)
        w = w_uk.double().permute(1, 0, 2).reshape(r_kv, g * d_h)
        for b, n in enumerate(lens):
            if n == 0:
                continue
            ids = table[b, : need[b]].long().cuda()
            c = pool[ids].reshape(-1, r_kv + d_r)[:n, :r_kv].double()
            got = keys[ids].reshape(-1, g * d_h)[:n].double()
            ref = c @ w
            # one rounding to bf16 (half of 2^-8 of the value) and fp32 sums of 512 products
            assert bool(((got - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-4).all()), "sequence %d" % b
