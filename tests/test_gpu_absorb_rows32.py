"""The absorb decode with one workgroup per 32 query rows, at the edges of its row blocks, pairs of tiles and chunks: 1 to 128
rows (blocks that end inside), chunks of one tile to many pairs, whole and half (the ring of two pairs fills, wraps and
drains), a last tile with one token, pages of several pairs, and logits that make a row's maximum move in every tile (the
eight waves then rescale together).  33 to 64 rows beyond one round of workgroups (num_cus = 1) take the general kernel.
Bar as everywhere: 2e-2 absolute, 1e-2 relative."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from oracle import gqla_oracle as O
from test_gpu_parity import Case, check, host, run_absorb_path

pytestmark = pytest.mark.gpu


def _case(h_q, g, s_q, lens, cp, num_cus, **kw):
    cfg = S.CONFIGS["C3"].with_(B=len(lens), h_q=h_q, g=g, s_q=s_q, L=0, paged=True, seed=93, **kw)
    print("rows32", h_q, g, s_q, lens, cp, num_cus, flush=True)
    return Case(cfg, lens=lens, chunk_pages=(cp, cp), num_cus=num_cus)


@pytest.mark.parametrize("h_q,g,s_q,lens,cp,num_cus", [
    (1, 1, 1, [1, 33, 64], 1, 256),                       # one row
    (16, 1, 2, [2, 31, 32, 33, 65, 97, 129], 8, 256),     # 32 rows; one to five tiles in a chunk
    (20, 4, 1, [700, 1], 3, 256),                         # 20 rows of 32
    (20, 5, 2, [65, 700, 2], 2, 1),                       # 40 rows, general kernel
    (20, 5, 2, [65, 700, 2], 2, 256),                     # 40 rows: the second block ends after 8
    (32, 8, 2, [1030, 64, 31, 129], 17, 256),             # 64 rows, 33 tiles in a chunk
    (64, 8, 1, [33, 65, 97, 257], 1, 256),                # 64 rows, chunks of one and two tiles
    (33, 1, 1, [161], 2, 256),                            # one row in the second block
    (128, 8, 1, [1000], 2, 256),                          # four workgroups of 32 rows a chunk
    (80, 8, 1, [300, 70], 2, 256),                        # the third ends after 16 rows
])
def test_rows_tiles_and_chunks(h_q, g, s_q, lens, cp, num_cus):
    case = _case(h_q, g, s_q, lens, cp, num_cus)
    try:
        run_absorb_path(case)
    finally:
        case.close()


def test_pages_of_several_pairs():
    case = _case(16, 1, 1, [256, 193, 500, 40], 1, 256, page_size=256)
    try:
        run_absorb_path(case)
    finally:
        case.close()


@pytest.mark.parametrize("h_q,g,num_cus", [(16, 1, 256), (64, 8, 256), (64, 8, 1)])
def test_maximum_moves_in_every_tile(h_q, g, num_cus):
    """k_R of tile i grows along a fixed direction that all queries share: each tile's logits exceed the last ones by 12 or
    more in base 2, past the threshold of 8.  The output is then close to the last tile's average, as in the oracle."""
    case = _case(h_q, g, 1, [32 * 6, 32 * 5 + 9], 64, num_cus)
    try:
        cfg = case.cfg
        dq = np.zeros_like(case.q_r)
        dq[..., 0] = 16.0
        case.q_r = S.quantize(case.q_r * 0.25 + dq, cfg.dtype)
        for b, L in enumerate(case.lens):
            rows = case.rows[b].copy()
            rows[:, cfg.r_kv] = (np.arange(L) // 32) * 8.0      # adds 16 * 8 / sqrt(192) = 9.2 per tile: 13.3 in base 2
            case.rows[b] = S.quantize(rows, cfg.dtype)
        from paper_2605_15250_amd.harness import build_latent_pool
        case.dec.latent_pool = build_latent_pool(cfg, case.lens, case.table, case.num_pages, lambda b, L: case.rows[b])
        q_hat = case.dec.absorb_query(case.d_q_c, case.d_w_uk)
        out, lse = case.dec.decode_absorb(q_hat, case.to_device(case.q_r, cfg.dtype), case.d_w_uv)
        torch.cuda.synchronize()
        for b in range(cfg.B):
            ref_o, ref_l = O.decode_absorb(host(q_hat)[b], case.q_r[b], case.c(b), case.kR(b), case.w_uv, d_h=cfg.d_h)
            check("out seq %d" % b, host(out)[b], ref_o, cfg.dtype)
            check("lse seq %d" % b, host(lse)[b], ref_l, cfg.dtype)
    finally:
        case.close()
