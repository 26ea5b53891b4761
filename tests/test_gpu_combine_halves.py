"""The merge with W_UV where a workgroup projects onto half of 128 value dims (few blocks of rows): one row per group up to the
edge where all 128 stay together (n_blocks * groups * value dims / 64 = 256), and value dims of 256.  Bar as everywhere: 2e-2
absolute, 1e-2 relative."""
import pytest

import synth_inputs as S
from test_gpu_parity import Case, run_absorb_path

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,g,s_q,d_h,d_v,lens", [
    (1, 1, 1, 128, 0, [300]),                        # one block with one row
    (128, 8, 1, 128, 0, [700]),                      # 4 rows a block, 64 workgroups
    (128, 8, 2, 128, 0, [130, 65, 40]),              # 12 blocks of 8 rows a group, 192 workgroups
    (64, 8, 2, 128, 0, [100] * 8),                   # 16 blocks of 8 rows, 256 workgroups: the last with halves
    (64, 8, 2, 128, 0, [100] * 9),                   # 18 blocks: 128 dims together
    (20, 4, 2, 192, 256, [90, 200]),                 # four halves of 256 value dims
    # the halves of a block go to ids equal modulo 8: workgroups per half not a multiple of 8, the grid filled up
    (54, 3, 2, 128, 0, [300, 70, 2, 130]),           # 108 and 4 empty ones
    (18, 1, 2, 128, 0, [500]),                       # 9 and 7
    (20, 5, 1, 192, 256, [130, 64, 3]),              # four quarters, 15 and 1
    (30, 15, 1, 192, 256, [200] * 9),                # both 128s, 75 and 5
    (20, 5, 2, 192, 256, [40] * 60),                 # 60 blocks a group in 25 workgroups, 125 and 3
])
def test_halves(h_q, g, s_q, d_h, d_v, lens):
    cfg = S.CONFIGS["C3"].with_(B=len(lens), h_q=h_q, g=g, s_q=s_q, L=0, paged=True, seed=98, d_h=d_h, d_v=d_v)
    print("combine halves", h_q, g, s_q, d_v, lens, flush=True)
    case = Case(cfg, lens=lens)
    try:
        run_absorb_path(case)
    finally:
        case.close()
