"""The merge of the chunk partials on both paths, at the edges of its launch shapes: one chunk, batches that end in the
middle, chains far longer than a batch, few rows (sliced chains), more row blocks than workgroups, ragged batches whose
sequences need different numbers of batches.  The oracle sees the same inputs; with one-page chunks (override 1) the
lengths choose the number of partials."""
import numpy as np
import pytest
import synth_inputs as S
from test_gpu_parity import Case, run_absorb_path, run_gqa_path

pytestmark = pytest.mark.gpu

P = 64


@pytest.mark.parametrize("h_q,g,s_q,lens", [
    (128, 8, 1, [P * 32 + 1]),                          # 33 chunks over 8 slices of the absorb merge: one batch and one chunk
    (128, 8, 2, [5, P * 70, P * 3 + 7]),                # 1, 70 and 4 chunks
    (16, 1, 2, [P * 9, 2, P * 8, P * 65]),              # one group, 32 rows
    (20, 4, 1, [P * 33 + 60, P * 17]),                  # 20 rows of 32: lanes without a row
    (64, 8, 1, [P * k + 3 for k in range(1, 30)]),      # mixed batches inside a block of rows
    (128, 8, 2, [70 + 40 * (k % 9) for k in range(40)]),  # 320 blocks of 32 rows: two per workgroup
    (128, 8, 1, [P * 4 + k for k in range(4)] * 16),    # 256 row blocks on the GQA path, four to five chunks each
    (128, 8, 1, [P * 12 + k for k in range(4)] * 4),    # 64 row blocks, 12 to 13 chunks: long chains, but workgroups enough without slices
    (128, 8, 1, [P * 12 + k for k in range(15)]),       # 60: slices
])
def test_merge_of_one_page_chunks(h_q, g, s_q, lens):
    cfg = S.CONFIGS["C3"].with_(B=len(lens), h_q=h_q, g=g, s_q=s_q, L=0, paged=True, seed=91)
    case = Case(cfg, lens=lens, chunk_pages=(1, 1))
    seqs = sorted({0, 1 % len(lens), len(lens) // 2, len(lens) - 1})
    try:
        print("combine", h_q, g, s_q, len(lens), flush=True)
        run_absorb_path(case, seqs)
        run_gqa_path(case, seqs)
    finally:
        case.close()


@pytest.mark.parametrize("lens", [[P * 40 + 9, 3], [100 + 10 * k for k in range(70)]])
def test_merge_with_a_value_dim_of_its_own(lens):
    cfg = S.CONFIGS["C3"].with_(B=len(lens), h_q=20, g=4, d_h=192, d_v=256, s_q=2, L=0, paged=True, seed=92)
    case = Case(cfg, lens=lens, chunk_pages=(1, 1))
    seqs = sorted({0, 1, len(lens) - 1})
    try:
        print("combine 192/256", len(lens), flush=True)
        run_absorb_path(case, seqs)
        run_gqa_path(case, seqs)
    finally:
        case.close()
