"""The two decode kernels over the 8-bit latent cache at the edges of their row blocks, tiles and chunks: row counts that end
inside a block (128 rows; with 32 and fewer, or few chunks, 32) and inside a wave's rows, chunks of one tile to many (the rings
of four tiles and of three pairs fill, wrap and drain), a last tile with one token, pages of several tiles, and logits that
make a row's maximum move in every tile (all waves then rescale together).  num_cus = 1 sends more than 32 rows to the kernel
for blocks of 128.  Same codes on both sides, so the plain 16-bit bar: 2e-2 absolute, 1e-2 relative."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from oracle import fp8_cache as F8
from oracle import gqla_oracle as O
from test_gpu_fp8_latent import _decode_and_check, _oracle_pool
from test_gpu_parity import Case, check, host

pytestmark = pytest.mark.gpu


def _case(h_q, g, s_q, lens, cp, num_cus=1, **kw):
    cfg = S.CONFIGS["C2"].with_(B=len(lens), h_q=h_q, g=g, s_q=s_q, L=0, paged=True, seed=97, **kw)
    print("fp8 rows", h_q, g, s_q, lens, cp, num_cus, flush=True)
    return Case(cfg, lens=lens, chunk_pages=(cp, cp), num_cus=num_cus)


@pytest.mark.parametrize("h_q,g,s_q,lens,cp,c_scale,num_cus", [
    (33, 1, 1, [161, 1], 2, 0.5, 1),                       # one row in the second wave
    (20, 5, 2, [65, 700, 2], 2, 0.37, 1),                  # 40 rows, two step tokens
    (64, 8, 1, [33, 65, 97, 129, 257], 1, 1.0, 1),         # 64 rows: the last two waves without rows; chunks of one and two tiles
    (128, 8, 1, [1, 31, 32, 96, 97, 1000], 16, 0.75, 1),   # one to 32 tiles in a chunk
    (80, 8, 2, [300, 70], 3, 0.02, 1),                     # 160 rows: a second block of 32; part of the latent saturates
    (132, 4, 1, [130, 64], 1, 2.5, 1),                     # four rows in the second block
    (1, 1, 1, [1, 33, 64], 1, 0.5, 256),                     # one row
    (16, 1, 2, [2, 31, 32, 33, 65, 97, 129, 161, 193, 225, 417], 8, 0.37, 256),   # 32 rows; one to 14 tiles in a chunk
    (20, 4, 1, [700, 1], 3, 1.0, 256),                       # 20 rows of 32
    (80, 8, 1, [300, 70], 2, 0.02, 256),                     # the third block ends after 16 rows
    (128, 8, 1, [1000], 4, 2.5, 256),                        # four workgroups of 32 rows a chunk
])
def test_rows_tiles_and_chunks(h_q, g, s_q, lens, cp, c_scale, num_cus):
    case = _case(h_q, g, s_q, lens, cp, num_cus)
    try:
        codes, pool = _oracle_pool(case, c_scale, fill=0xFF)      # slots no token owns: NaN codes
        case.dec.latent_fp8_pool = torch.from_numpy(pool).cuda()
        _decode_and_check(case, c_scale, codes, "decode_absorb_fp8")
    finally:
        case.close()


@pytest.mark.parametrize("h_q,num_cus", [(128, 1), (16, 256)])
def test_pages_of_several_tiles(h_q, num_cus):
    case = _case(h_q, 8, 1, [256, 193, 500, 40], 1, num_cus, page_size=256)
    try:
        codes, pool = _oracle_pool(case, 0.5)
        case.dec.latent_fp8_pool = torch.from_numpy(pool).cuda()
        _decode_and_check(case, 0.5, codes, "decode_absorb_fp8")
    finally:
        case.close()


@pytest.mark.parametrize("h_q,num_cus", [(64, 1), (128, 1), (16, 256)])
def test_maximum_moves_in_every_tile(h_q, num_cus):
    """k_R of tile i grows along a fixed direction that all queries share: each tile's logits exceed the last ones by 12 or
    more in base 2, past the threshold of 8."""
    case = _case(h_q, 8, 1, [32 * 6, 32 * 5 + 9], 64, num_cus)
    try:
        cfg, dec = case.cfg, case.dec
        dq = np.zeros_like(case.q_r)
        dq[..., 0] = 16.0
        case.q_r = S.quantize(case.q_r * 0.25 + dq, cfg.dtype)
        for b, L in enumerate(case.lens):
            rows = case.rows[b].copy()
            rows[:, cfg.r_kv] = (np.arange(L) // 32) * 8.0      # adds 16 * 8 / sqrt(192) = 9.2 per tile: 13.3 in base 2
            case.rows[b] = S.quantize(rows, cfg.dtype)
        codes, pool = _oracle_pool(case, 0.5)
        dec.latent_fp8_pool = torch.from_numpy(pool).cuda()
        q_hat = dec.absorb_query(case.d_q_c, case.d_w_uk)
        out, lse = dec.decode_absorb_fp8(q_hat, case.to_device(case.q_r, cfg.dtype), 0.5, case.d_w_uv)
        torch.cuda.synchronize()
        for b in range(cfg.B):
            c_deq = F8.dequantize_e4m3(codes[b]) * 0.5
            ref_o, ref_l = O.decode_absorb(host(q_hat)[b], case.q_r[b], c_deq, case.kR(b), case.w_uv, d_h=cfg.d_h)
            check("out seq %d" % b, host(out)[b], ref_o, cfg.dtype)
            check("lse seq %d" % b, host(lse)[b], ref_l, cfg.dtype)
    finally:
        case.close()
