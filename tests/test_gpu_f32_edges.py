"""The fp32 kernels where their sharing out of sums over 256 threads changes: fewer and more units than threads, one and
several passes of 64 tokens, one chunk per sequence (the decode writes the output itself) and several (partials and a
merge), column blocks that end inside a wave, pages of 8.  Bars as for every fp32 shape: 1e-4 absolute, 1e-5 relative."""
import pytest
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
