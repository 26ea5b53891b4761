"""The GQA decode over the 8-bit cache, chunks of one to seven tiles in each form of the kernel -- k_R shared by all waves of a
workgroup, by those of a row block, not at all (three, five groups), token teams, two row blocks a wave -- and the form that keeps
two tiles of codes in flight (groups a multiple of eight, chunks of at least four tiles and more than half as many as a group has rows:
either side of those lines, and sequences of one tile to the whole chunk, last pairs with and without a second tile) -- with NaN codes in
every byte that no token owns, and with a page id out of range (its tokens count as absent).  Bars as everywhere."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from oracle import fp8_cache as F8
from oracle import gqla_oracle as O
from test_gpu_fp8_cache import _bf16_bits
from test_gpu_parity import Case, check, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,g,s_q,lens,cp,num_cus,lost", [
    (128, 8, 2, [2, 32, 33, 64, 65, 97, 129, 161, 200], 4, 1, None),   # one to seven tiles, k_R shared by eight groups
    (128, 8, 1, [400, 190], 1, 1, None),                               # chunks of one page: one pair, or one tile
    (64, 8, 2, [300, 129], 8, 1, 1),                                   # the second page of each sequence is lost
    (48, 3, 1, [2, 40, 65, 97, 130, 200], 4, 1, None),                 # three groups: teams of one
    (40, 5, 2, [300, 129], 8, 256, 1),                                 # five: teams
    (64, 4, 2, [65, 97, 200], 4, 1, None),                             # workgroups of four waves
    (32, 2, 2, [65, 97, 200], 4, 1, None),                             # of two
    (16, 1, 2, [33, 300, 900], 8, 256, None),                          # one group: teams of eight, waves with no, one, two tiles
    (128, 4, 2, [33, 65, 97, 200], 4, 1, None),                        # two row blocks a wave
    (120, 3, 1, [33, 65, 97, 200], 4, 1, 1),                           # the same, k_R not shared
    (56, 8, 1, [1, 32, 33, 64, 65, 97, 128, 300], 2, 1, None),         # 7 rows, four tiles: two in flight
    (64, 8, 1, [1, 33, 64, 130, 300], 2, 1, None),                     # 8 rows: one
    (128, 8, 1, [1, 33, 64, 130, 225, 320, 600], 5, 1, None),          # 16 rows, ten tiles: two
    (128, 8, 1, [33, 161, 256, 400], 4, 1, None),                      # eight: one
    (128, 8, 2, [2, 33, 64, 290, 545, 576, 700], 9, 1, None),          # 32 rows, eighteen tiles: two
    (128, 8, 2, [33, 417, 512, 700], 8, 1, None),                      # sixteen: one
    (48, 16, 1, [33, 200, 129], 4, 1, 1),                              # 16 groups, two in flight, the second page of each sequence lost
])
def test_fp8_tiles(h_q, g, s_q, lens, cp, num_cus, lost):
    print("fp8 tiles", h_q, g, s_q, lens, cp, num_cus, lost, flush=True)
    cfg = S.CONFIGS["C2"].with_(B=len(lens), h_q=h_q, g=g, s_q=s_q, L=0, paged=True, seed=910 + h_q)
    case = Case(cfg, lens=lens, chunk_pages=(0, cp), num_cus=num_cus)
    dec = case.dec
    ks, vs = 0.5, 2.0
    try:
        KCq, Vq, kR = [], [], [case.kR(b) for b in range(cfg.B)]
        for b in range(cfg.B):
            KC, V = O.expand_latent(case.c(b), case.w_uk, case.w_uv)
            KCq.append(F8.quantize_tensor(S.quantize(KC, cfg.dtype), ks)); Vq.append(F8.quantize_tensor(S.quantize(V, cfg.dtype), vs))
        pool = F8.pack_fp8_pool(KCq, Vq, [_bf16_bits(x) for x in kR], case.table, case.num_pages, cfg.page_size, fill=0x7F)
        dec.alloc_expanded_fp8(fill=0x7F)
        dec.expanded_fp8_pool = torch.from_numpy(pool).cuda()
        keep = [np.ones(int(n), bool) for n in lens]
        if lost is not None:
            dec.d_table[:, lost] = case.num_pages
            for k in keep:
                k[lost * cfg.page_size:(lost + 1) * cfg.page_size] = False
        out, lse = dec.decode_gqa_fp8(case.d_q_c, case.d_q_r, ks, vs)
        torch.cuda.synchronize()
        ref_o, ref_l = [], []
        for b in range(cfg.B):
            K, V = F8.dequantize_e4m3(KCq[b]) * ks, F8.dequantize_e4m3(Vq[b]) * vs
            axis = [i for i, n in enumerate(K.shape) if n == lens[b]][0]
            o, l = O.decode_gqa(case.q_c[b], case.q_r[b], np.compress(keep[b], K, axis), np.compress(keep[b], V, axis), kR[b][keep[b]])
            ref_o.append(o); ref_l.append(l)
        check("decode_gqa_fp8", host(out), np.stack(ref_o), cfg.dtype)
        check("decode_gqa_fp8 lse", host(lse), np.stack(ref_l), cfg.dtype)
    finally:
        case.close()
