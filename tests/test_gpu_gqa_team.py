"""The GQA decode with two, four or eight waves per (chunk, group), chosen from the plan and num_cus: chunks with fewer tiles
than the team's waves would have (the ragged last chunk of a sequence), more than two tiles a wave, teams that do not fill the
last workgroup, workgroups of one and of several teams, rows that end inside a block, both pairs of dims and the 8-bit cache (through test_gpu_fp8_cache's own cases).
Bars as everywhere."""
import pytest
import synth_inputs as S
from test_gpu_parity import Case, run_gqa_path

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,g,s_q,d_h,d_v,lens,cp,num_cus", [
    (128, 8, 1, 128, 128, [300], 2, 256),             # 24 items, teams of four; the last chunk has two tiles
    (128, 8, 2, 128, 128, [1030, 2], 8, 256),         # teams of eight, two tiles a wave and one token in the last
    (48, 3, 1, 128, 128, [200, 65], 1, 256),          # teams of two: 15 items, half of the last workgroup repeats
    (24, 3, 2, 128, 128, [500], 3, 20),               # 9 items, teams of four over 20 units' waves
    (64, 8, 1, 128, 128, [130, 700, 1], 4, 40),       # 40 items on 40 units: eight waves each
    (64, 8, 1, 128, 128, [130, 700, 1], 4, 39),       # one unit less: four
    (20, 4, 2, 192, 256, [129, 900, 2], 3, 256),      # (192, 256): up to four
    (20, 5, 1, 192, 256, [129, 64], 1, 256),          # teams of two, 15 items
    # a workgroup of one team while there are no more of them than units; several teams, some of them spare, beyond
    (128, 8, 1, 128, 128, [300], 2, 24),              # 24 items, teams of four, 24 units: one team per workgroup
    (128, 8, 1, 128, 128, [300], 2, 23),              # 23 units: two
    (48, 3, 1, 128, 128, [200, 65], 1, 5),            # 15 items, teams of two, 5 units: four teams per workgroup, one spare
    (20, 5, 1, 192, 256, [129, 64], 1, 8),            # (192, 256): 15 items, 8 units: two, one spare
    (64, 4, 2, 128, 128, [130, 2], 1, 256),           # four groups, chunks of one page: teams of two
    (64, 4, 2, 128, 128, [130, 2], 1, 7),             # 16 items, half of 7 units' waves: none
    (32, 2, 2, 128, 128, [130, 64], 1, 256),          # two groups, chunks of one page: none
    (32, 2, 2, 128, 128, [130, 300], 2, 256),         # of two pages: teams of four
])
def test_token_teams(h_q, g, s_q, d_h, d_v, lens, cp, num_cus):
    cfg = S.CONFIGS["C3"].with_(B=len(lens), h_q=h_q, g=g, s_q=s_q, d_h=d_h, d_v=d_v, L=0, paged=True, seed=95)
    print("team", h_q, g, s_q, d_h, lens, cp, num_cus, flush=True)
    case = Case(cfg, lens=lens, chunk_pages=(cp, cp), num_cus=num_cus)
    try:
        run_gqa_path(case)
    finally:
        case.close()
