"""gqla_expand_cache when the token blocks exceed one round of 256 workgroups: blocks of whole rounds keep all groups, those of
an unfinished last round of at most 128 share theirs out.  One and two lengths-per-wave scans (40 and 70 sequences), last
rounds of 0, 1, 128 and 129 blocks; every byte against expanding the groups one by one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,last", [(40, 0), (40, 1), (70, 128), (70, 129), (70, 0)])
def test_last_round(nb, last):
    from paper_2605_15250_amd import binding as B
    g, d, r_kv, d_r, P = 3, 128, 512, 64, 64
    blocks = [(256 + last) // nb + (1 if i < (256 + last) % nb else 0) for i in range(nb)]
    lens = [256 * n - (37 * i) % 256 for i, n in enumerate(blocks)]          # ragged ends, the same number of blocks
    max_pages = max(-(-n // P) for n in lens)
    gen = torch.Generator(device="cuda").manual_seed(9)
    pool = torch.randn(nb * max_pages, P, r_kv + d_r, generator=gen, device="cuda").bfloat16()
    w_uk = (torch.randn(g, r_kv, d, generator=gen, device="cuda") * r_kv ** -0.5).bfloat16()
    w_uv = (torch.randn(g, r_kv, d, generator=gen, device="cuda") * r_kv ** -0.5).bfloat16()
    d_lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    shape = B.make_shape(nb, g, g, d, r_kv, d_r, 1, B.GQLA_BF16)
    ws = torch.empty(B.gqla_expand_workspace_bytes(shape, g), dtype=torch.uint8, device="cuda")
    latent = B.make_cache(pool, d_lens, None, P, max_pages, nb * max_pages)

    def expand(begin, count):
        out = torch.full((nb * max_pages, P * (2 * count * d + d_r)), 7.0, dtype=torch.bfloat16, device="cuda")
        print("expand", nb, last, begin, count, flush=True)
        B.gqla_expand_cache(shape, latent, w_uk, w_uv, begin, count, B.make_cache(out, d_lens, None, P, max_pages, nb * max_pages, count), ws)
        torch.cuda.synchronize()
        return out
    full, n = expand(0, g), P * d
    for j in range(g):
        one = expand(j, 1)
        assert torch.equal(full[:, j * n:(j + 1) * n], one[:, :n]) and torch.equal(full[:, (g + j) * n:(g + j + 1) * n], one[:, n:2 * n]), j
        assert torch.equal(full[:, 2 * g * n:], one[:, 2 * n:])
    c = pool[0, :, :r_kv].float()
    keys = full[0, :n].float().reshape(d // 8, P, 8).permute(1, 0, 2).reshape(P, d)
    ref = c @ w_uk[0].float()
    assert bool(((keys - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-4).all())
