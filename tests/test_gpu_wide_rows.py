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
    shape = B.make_shape(nb, G, G, D, R_KV, D_R, 1, B.GQLA_BF16)

    def values(*size):
        return torch.randn(*size, generator=gen, device="cuda").bfloat16()

    def cache(pool, groups=0):
        return B.make_cache(pool, d_lens, d_table, P, max_pages, num_pages, groups)
    latent, keys = values(num_pages, P * (R_KV + D_R)), values(num_pages, P * (2 * G * D + D_R))
    w_uk, w_uv, w_inv = values(G, R_KV, D), values(G, R_KV, D), values(R_KV, G * D)
    ws = torch.empty(B.gqla_expand_workspace_bytes(shape, G), dtype=torch.uint8, device="cuda")
    print(op, nb, max_pages, flush=True)
    if op == "expand":
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


@pytest.mark.parametrize("op,nb", [("expand", 1), ("expand_fp8", 1)])
def test_row_of_two_to_the_31_tokens(op, nb):
    narrow = _switch(op, nb, 2)
    assert int((narrow != 0).sum()) > 0
    assert torch.equal(_switch(op, nb, 1 << 21), narrow)
