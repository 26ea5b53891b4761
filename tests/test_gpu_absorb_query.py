"""Query absorption where its launch changes: the latent dims in 4, 2 or 1 shares, workgroups that walk over several row
blocks, row counts that end inside a block.  Reference: fp32 products of the same bits; the result is rounded once to bf16
(2^-9 relative) and summed in fp32 (128 products of order 1/sqrt(512): below 1e-6), so 2^-8 relative + 1e-5 is the bar."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,g,rows", [
    (8, 8, 1),        # one row per group
    (128, 8, 1), (128, 8, 3),
    (128, 8, 16),     # 8 blocks x 8 groups: 4 shares, all units
    (128, 8, 17),     # 2 shares, the last block half full
    (128, 8, 33),     # 1 share
    (128, 8, 67),     # 34 blocks over 32 workgroups a group
    (128, 4, 100),    # 100 blocks over 64
    (16, 1, 521),     # 261 blocks over 256, one group
    (96, 3, 7),
])
def test_absorb_query_launch_edges(h_q, g, rows):
    from paper_2605_15250_amd import binding as B
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q = torch.empty(rows, 1, h_q, 128, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    w = torch.empty(g, 512, 128, dtype=torch.bfloat16, device="cuda").normal_(0.0, 512 ** -0.5, generator=gen)
    out = torch.full((rows + 1, 1, h_q, 512), float("nan"), dtype=torch.bfloat16, device="cuda")
    print("absorb_query", h_q, g, rows, flush=True)
    B.gqla_absorb_query(B.make_shape(rows, h_q, g, 128, 512, 64, 1, B.GQLA_BF16), q, w, out)
    torch.cuda.synchronize()
    G = h_q // g
    for j in range(g):
        ref = q[:, 0, j * G:(j + 1) * G].float().reshape(-1, 128) @ w[j].float().T.contiguous()
        got = out[:rows, 0, j * G:(j + 1) * G].float().reshape(-1, 512)
        assert bool(((got - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-5).all()), j
    assert bool(torch.isnan(out[rows]).all())     # nothing behind the last row
