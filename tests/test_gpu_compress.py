"""gqla_compress_cache at the edges of its kernel: token counts around the 64-token halves and the 128-token tiles, more
sequences than one scan of the lengths covers, and the shortest contractions.
Reference: fp64 product of the same bf16 values."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EDGES = [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257]


@pytest.mark.parametrize("g,d_h,d_v,lens,page_size,paged", [
    (4, 128, 128, EDGES, 64, True),                    # eight stages of the contraction, the fewest
    (3, 192, 256, EDGES[:6], 128, True),               # nine
    (5, 128, 128, [130], 64, False),
    (8, 128, 128, [1, 0, 200, 0, 129] + [3] * 60 + [0, 64, 65], 64, True),   # 68 sequences, some empty
])
def test_compress_edges(g, d_h, d_v, lens, page_size, paged):
    from paper_2605_15250_amd import binding as B
    r_kv, d_r, P = 512, 64, page_size
    gen = torch.Generator(device="cuda").manual_seed(77)
    nb, npages = len(lens), [-(-n // P) for n in lens]
    max_pages = max(npages) + 1                        # (one page of the row that no sequence reaches)
    num_pages = nb * max_pages
    order = torch.randperm(num_pages, generator=gen, device="cuda").cpu().numpy() if paged else np.arange(num_pages)
    table = order.reshape(nb, max_pages).astype(np.int32)
    K = g * d_h
    pool = torch.randn(num_pages, P * (g * (d_h + d_v) + d_r), generator=gen, device="cuda").bfloat16()
    w_inv = (torch.randn(r_kv, K, generator=gen, device="cuda") * K ** -0.5).bfloat16()
    latent = torch.full((num_pages, P, r_kv + d_r), float("nan"), dtype=torch.bfloat16, device="cuda")
    d_lens, d_table = torch.tensor(lens, dtype=torch.int32, device="cuda"), torch.from_numpy(table).cuda()
    shape = B.make_shape(nb, g * 4, g, d_h, r_kv, d_r, 1, B.GQLA_BF16, 0.0, d_v)
    tab = d_table if paged else None
    print("compress", g, d_h, nb, flush=True)
    B.gqla_compress_cache(shape, B.make_cache(pool, d_lens, tab, P, max_pages, num_pages, g), w_inv,
                          B.make_cache(latent, d_lens, tab, P, max_pages, num_pages))
    torch.cuda.synchronize()
    got = latent.float().cpu()
    assert int(torch.isnan(got).sum()) == got.numel() - sum(lens) * (r_kv + d_r), "only the tokens' rows are written"
    for b, n in enumerate(lens):
        if n == 0:
            continue
        ids = torch.from_numpy(table[b, : npages[b]].astype(np.int64))
        pages = pool.cpu()[ids]
        keys = pages[:, : g * P * d_h].reshape(-1, K // 8, P, 8).permute(0, 2, 1, 3).reshape(-1, K)[:n].double()
        k_r = pages[:, g * P * (d_h + d_v):].reshape(-1, d_r // 8, P, 8).permute(0, 2, 1, 3).reshape(-1, d_r)[:n]
        rows = got[ids].reshape(-1, r_kv + d_r)[:n]
        ref = keys @ w_inv.cpu().double().T
        # one rounding to bf16 (2^-9 of the value) and fp32 sums of K products of magnitude ~K^-1/2 (K 2^-24 of their sum)
        bound = ref.abs() * 2.0 ** -8 + 1e-4
        assert bool(((rows[:, :r_kv].double() - ref).abs() <= bound).all()), "sequence %d (%d tokens)" % (b, n)
        assert torch.equal(rows[:, r_kv:], k_r.float()), "k_R is copied"
