"""The fp32 kernels where their sharing out of sums over 256 threads changes: fewer and more units than threads, one and
several passes of 64 tokens, one chunk per sequence (the decode writes the output itself) and several (partials and a
merge), column blocks that end inside a wave, pages of 8.  Bars as for every fp32 shape: 1e-4 absolute, 1e-5 relative."""
import pytest
import torch

import synth_inputs as S
from test_gpu_parity import Case, run_absorb_path, run_gqa_path

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,g,s_q,d_h,d_v,r_kv,d_r,page,lens,cp", [
    (2, 1, 1, 8, 8, 8, 8, 8, [1], 1),                          # smallest dims, one token
    (8, 2, 1, 16, 16, 32, 8, 16, [64, 63, 65], 64),            # one chunk each: a pass of 64, one short of it, one beyond
    (8, 2, 2, 16, 16, 32, 8, 16, [64, 2, 161], 2),             # several chunks
    (6, 3, 2, 24, 40, 72, 24, 24, [190, 25], 8),               # dims that divide nothing evenly, ragged page ends
    (4, 4, 1, 64, 64, 128, 32, 16, [1000], 64),                # sixteen passes in one chunk
    (4, 1, 1, 512, 264, 512, 72, 8, [77, 9], 3),               # widest: more units than threads
    (2, 2, 2, 72, 512, 264, 8, 8, [130], 64),                  # the same, one chunk
])
def test_fp32_edges(h_q, g, s_q, d_h, d_v, r_kv, d_r, page, lens, cp):
    cfg = S.CONFIGS["C0"].with_(B=len(lens), h_q=h_q, g=g, s_q=s_q, d_h=d_h, d_v=d_v, r_kv=r_kv, d_r=d_r, page_size=page, L=0,
                                paged=True, seed=78)
    print("fp32", cfg, lens, cp, flush=True)
    case = Case(cfg, lens=lens, chunk_pages=(cp, cp))
    try:
        run_absorb_path(case)
        run_gqa_path(case)
    finally:
        case.close()


@pytest.mark.parametrize("lens", [[8192, 8193, 20011], [7]])
def test_f32_expansion_of_more_eights_than_workgroups(lens):
    """Beyond 8192 tokens of a row a workgroup takes several groups of eight tokens in turn.  Against the fp64 product."""
    from paper_2605_15250_amd import binding as B
    g, d, r_kv, d_r, P = 2, 8, 16, 8, 16
    nb, max_pages = len(lens), 20016 // P
    gen = torch.Generator(device="cuda").manual_seed(6)
    pool = torch.randn(nb * max_pages, P, r_kv + d_r, generator=gen, device="cuda")
    w_uk, w_uv = (torch.randn(g, r_kv, d, generator=gen, device="cuda") for _ in range(2))
    d_lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    out = torch.full((nb * max_pages, P * (2 * g * d + d_r)), float("nan"), device="cuda")
    shape = B.make_shape(nb, g, g, d, r_kv, d_r, 1, B.GQLA_F32)
    print("expand f32", lens, flush=True)
    B.gqla_expand_cache(shape, B.make_cache(pool, d_lens, None, P, max_pages, nb * max_pages), w_uk, w_uv, 0, g,
                        B.make_cache(out, d_lens, None, P, max_pages, nb * max_pages, g))
    torch.cuda.synchronize()
    n = g * P * d
    keys = out[:, :n].reshape(-1, g, P, 8).transpose(1, 2).reshape(nb, max_pages * P, g * d)
    vals = out[:, n:2 * n].reshape(-1, g, P // 8, d, 8).permute(0, 2, 4, 1, 3).reshape(nb, max_pages * P, g * d)
    rope = out[:, 2 * n:].reshape(nb, max_pages * P, d_r)
    rows = pool.reshape(nb, max_pages * P, r_kv + d_r)
    for b, L in enumerate(lens):
        c = rows[b, :L, :r_kv].double()
        for got, w in ((keys, w_uk), (vals, w_uv)):
            ref = c @ w.double().permute(1, 0, 2).reshape(r_kv, g * d)
            assert float((got[b, :L].double() - ref).norm() / ref.norm()) < 1e-6      # fp32 sums of 16 products
            assert bool(got[b, L:].isnan().all())
        assert torch.equal(rope[b, :L], rows[b, :L, r_kv:]) and bool(rope[b, L:].isnan().all())


@pytest.mark.parametrize("path", ["absorb", "gqa"])
@pytest.mark.parametrize("cp", [0, 1])
def test_f32_output_laid_over_the_queries(path, cp):
    """The output may lie where the queries were (value dims other than the queries' make rows meet those of other heads and
    sequences), with one chunk per sequence and with several: the values of a call with an output of its own."""
    from paper_2605_15250_amd import binding as B
    g, h_q, d_h, d_v, r_kv, d_r, P, lens = 2, 32, 64, 16, 64, 8, 16, [100, 40, 77] * 20
    nb, max_pages = len(lens), 7
    gen = torch.Generator(device="cuda").manual_seed(8)
    absorb = path == "absorb"
    width = r_kv + d_r if absorb else g * (d_h + d_v) + d_r
    pool = torch.randn(nb * max_pages, P * width, generator=gen, device="cuda")
    q = torch.randn(nb, h_q, r_kv if absorb else d_h, generator=gen, device="cuda")
    q_r = torch.randn(nb, h_q, d_r, generator=gen, device="cuda")
    w_uv = torch.randn(g, r_kv, d_v, generator=gen, device="cuda")
    d_lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    shape = B.make_shape(nb, h_q, g, d_h, r_kv, d_r, 1, B.GQLA_F32, 0.0, d_v)
    cache = B.make_cache(pool, d_lens, None, P, max_pages, nb * max_pages, 0 if absorb else g)
    plan = B.gqla_plan_create(shape, lens, P, 256, B.GQLA_PATH_ABSORB if absorb else B.GQLA_PATH_GQA, cp or max_pages)
    assert (B.gqla_plan_num_chunks(plan) == nb) == (cp == 0)
    ws = torch.empty(B.gqla_plan_workspace_bytes(plan), dtype=torch.uint8, device="cuda")
    B.gqla_plan_upload(plan, ws)

    def decode(out, lse):
        print(path, cp, flush=True)
        if absorb:
            B.gqla_decode_absorb(shape, plan, q, q_r, cache, w_uv, out, lse, ws)
        else:
            B.gqla_decode_gqa(shape, plan, q, q_r, cache, out, lse, ws)
        torch.cuda.synchronize()
        return out.clone(), lse.clone()
    n = nb * h_q
    apart = decode(torch.empty(nb, h_q, d_v, device="cuda"), torch.empty(nb, h_q, device="cuda"))
    over = decode(q.view(-1)[:n * d_v].view(nb, h_q, d_v), q_r.view(-1)[:n].view(nb, h_q))
    B.gqla_plan_destroy(plan)
    # (a merge of one partial rounds its weight of 1 through an exponential and a logarithm: 2^-22)
    assert float((apart[0] - over[0]).abs().max()) <= 1e-6 * float(apart[0].abs().max())
    assert float((apart[1] - over[1]).abs().max()) <= 1e-5
