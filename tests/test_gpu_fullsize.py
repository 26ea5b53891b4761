"""GPU parity at the workload's full sizes, in the launch configuration bench.py times (default plans, 256 CUs).

The oracle cannot redo a whole configuration in seconds, so each test checks
  * sampled (sequence, group) slices element by element against the oracle (always the shortest and the longest
    sequence, and for the ragged configuration one whose length is not a multiple of the page size), and
  * properties that hold at any size over EVERY output: finiteness, and the paper's own invariant that the two
    decode paths agree (Sec. 3.1) -- here between two independent GPU kernels, within the bf16 tolerance.
Tolerances as in test_gpu_parity.py: max abs 2e-2, relative L2 1e-2."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from oracle import gqla_oracle as O

pytestmark = pytest.mark.gpu

MAX_ABS, REL_L2 = 2e-2, 1e-2


def rel_l2(a, ref):
    a = np.asarray(a, np.float64)
    ref = np.asarray(ref, np.float64)
    return float(np.linalg.norm(a - ref) / max(np.linalg.norm(ref), 1e-300))


def check(name, got, ref):
    got = np.asarray(got, np.float64)
    err = float(np.max(np.abs(got - ref)))
    r = rel_l2(got, ref)
    print("%-44s max_abs %.3e  rel_l2 %.3e" % (name, err, r), flush=True)
    assert np.isfinite(got).all(), name
    assert err <= MAX_ABS and r <= REL_L2, (name, err, r)


class FullCase:
    def __init__(self, cfg, groups=None, group_begin=0):
        from paper_2605_15250_amd.harness import Decoder, to_device, build_latent_pool
        self.cfg = cfg
        self.lens = S.seq_lens(cfg)
        self.table, self.num_pages = S.page_table(cfg, self.lens)
        self.w_uk, self.w_uv = S.weights(cfg)
        self.q_c, self.q_r = S.queries(cfg)
        self.dec = Decoder(cfg, self.lens, self.table, self.num_pages, groups=groups, group_begin=group_begin,
                           use_page_table=cfg.paged)
        print("building latent pool: %d sequences, %d tokens" % (cfg.B, int(self.lens.sum())), flush=True)
        self.dec.latent_pool = build_latent_pool(cfg, self.lens, self.table, self.num_pages,
                                                 lambda b, L: S.sequence_rows(cfg, b, L))
        self.d = lambda x: to_device(x, cfg.dtype)
        self.d_w_uk, self.d_w_uv = self.d(self.w_uk), self.d(self.w_uv)

    def rows(self, b):
        r = S.sequence_rows(self.cfg, b, self.lens[b])
        return r[:, :self.cfg.r_kv], r[:, self.cfg.r_kv:]

    def named_sequences(self):
        """the shortest, the longest, and one whose length is not a multiple of the page size"""
        picks = {int(np.argmin(self.lens)), int(np.argmax(self.lens))}
        odd = [b for b in range(self.cfg.B) if self.lens[b] % self.cfg.page_size and b not in picks]
        if odd:
            picks.add(odd[len(odd) // 2])
        return sorted(picks)

    def sample_sequences(self, n=0):
        """the named ones plus, up to n in all, sequences spread evenly over the batch"""
        picks = list(self.named_sequences())
        for b in np.linspace(0, self.cfg.B - 1, max(n, 0)).astype(int):
            if len(picks) >= n:
                break
            if int(b) not in picks:
                picks.append(int(b))
        return sorted(picks)

    def close(self):
        self.dec.close()


def cfg_page(case):
    return case.cfg.page_size


def oracle_group(case, b, j, path):
    """Oracle output of sequence b restricted to the heads of group j (a self-consistent h_q = G, g = 1 problem)."""
    cfg = case.cfg
    G = cfg.h_q // cfg.g
    hs = slice(j * G, (j + 1) * G)
    c, kR = case.rows(b)
    qc, qr = case.q_c[b][:, hs], case.q_r[b][:, hs]
    wk, wv = case.w_uk[j:j + 1], case.w_uv[j:j + 1]
    if path == "absorb":
        return O.decode_absorb(O.absorb_query(qc, wk), qr, c, kR, wv, d_h=cfg.d_h)
    KC, V = O.expand_latent(c, wk, wv)
    return O.decode_gqa(qc, qr, KC, V, kR)


def run_both_paths(case, groups_to_check, groups_named=None, n_seqs=0):
    groups_named = list(groups_to_check) if groups_named is None else list(groups_named)
    cfg = case.cfg
    G = cfg.h_q // cfg.g
    q_hat = case.dec.absorb_query(case.d(case.q_c), case.d_w_uk)
    out_a, lse_a = case.dec.decode_absorb(q_hat, case.d(case.q_r), case.d_w_uv)
    case.dec.alloc_expanded()
    case.dec.expand(case.d_w_uk, case.d_w_uv)
    out_g, lse_g = case.dec.decode_gqa(case.d(case.q_c), case.d(case.q_r))
    torch.cuda.synchronize()
    oa, og = out_a.float().cpu().numpy(), out_g.float().cpu().numpy()
    la, lg = lse_a.cpu().numpy(), lse_g.cpu().numpy()
    # properties over every output
    assert np.isfinite(oa).all() and np.isfinite(og).all() and np.isfinite(la).all() and np.isfinite(lg).all()
    check("absorb vs gqa path, all outputs", oa, og)
    assert float(np.max(np.abs(la - lg))) <= 2e-2, "lse of the two paths"
    # sampled slices against the oracle: every group in groups_named for the three named sequences, the groups in
    # groups_to_check for the rest of the sample; relative L2 is reported (and gated) per sequence as well
    named = case.named_sequences()
    per_seq = []
    for b in case.sample_sequences(n_seqs):
        ea = eg = na = 0.0
        for j in (groups_named if b in named else groups_to_check):
            hs = slice(j * G, (j + 1) * G)
            ref_o, ref_l = oracle_group(case, b, j, "absorb")
            check("absorb  b=%d L=%d group %d" % (b, case.lens[b], j), oa[b][:, hs], ref_o)
            check("gqa     b=%d L=%d group %d" % (b, case.lens[b], j), og[b][:, hs], ref_o)
            assert float(np.max(np.abs(la[b][:, hs] - ref_l))) <= 2e-2
            assert float(np.max(np.abs(lg[b][:, hs] - ref_l))) <= 2e-2
            ea += float(np.sum((oa[b][:, hs] - ref_o) ** 2))
            eg += float(np.sum((og[b][:, hs] - ref_o) ** 2))
            na += float(np.sum(ref_o ** 2))
        per_seq.append((b, int(case.lens[b]), (ea / na) ** 0.5, (eg / na) ** 0.5))
    print("per-sequence relative L2 (sequence, L, absorb, gqa):", flush=True)
    for b, L, ra, rg in per_seq:
        print("   b=%3d  L=%6d  absorb %.3e  gqa %.3e" % (b, L, ra, rg), flush=True)
        assert ra <= REL_L2 and rg <= REL_L2, (b, L, ra, rg)
    return per_seq


def test_c1_llama3_shape_both_paths():
    case = FullCase(S.CONFIGS["C1"])
    try:
        run_both_paths(case, groups_to_check=range(8))     # all 32 heads of the sampled sequences
    finally:
        case.close()


def test_c2_c3_canonical_both_paths_with_mtp():
    """The canonical absorb and GQA decodes share shape and weights; the s_q = 2 configuration exercises both paths (row 1 of the
    step is a plain s_q = 1 decode at length L, row 0 one at length L - 1)."""
    case = FullCase(S.CONFIGS["C3"])
    try:
        run_both_paths(case, groups_to_check=[0, 5])
    finally:
        case.close()


def test_c3_step_updates_and_fp8_cache_at_full_size():
    """The canonical GQA decode at full size: the per-step cache updates (append + tail expansion on top of a one-shot expansion of
    the prefix) must reproduce the one-shot expansion of everything bit for bit, and the decode over the 8-bit cache
    (expand -> quantise on the GPU) is checked on sampled (sequence, group) slices against the oracle's chain."""
    from oracle import fp8_cache as F8
    cfg = S.CONFIGS["C3"]
    case = FullCase(cfg)
    dec = case.dec
    try:
        G = cfg.h_q // cfg.g
        dec.alloc_expanded(fill=0.0)
        dec.expand(case.d_w_uk, case.d_w_uv)
        torch.cuda.synchronize()
        one_shot = dec.expanded_pool.clone()
        # the step's rows appended again (same values) and their positions expanded again into a zeroed copy of the tail
        W = cfg.r_kv + cfg.d_r
        flat = dec.latent_pool.view(-1, W)
        idx = []
        for b in range(cfg.B):
            for t in range(int(case.lens[b]) - cfg.s_q, int(case.lens[b])):
                idx.append(int(case.table[b][t // cfg.page_size]) * cfg.page_size + t % cfg.page_size)
        idx_t = torch.tensor(idx, device="cuda")
        rows = flat[idx_t].view(cfg.B, cfg.s_q, W).contiguous()
        flat[idx_t] = 0
        dec.append_latent(rows)
        dec.expand_tail(case.d_w_uk, case.d_w_uv, cfg.s_q)
        torch.cuda.synchronize()
        assert torch.equal(dec.expanded_pool.view(torch.int16), one_shot.view(torch.int16)), "tail expansion vs one-shot expansion"
        # the same from weights repacked ahead of time (what the benchmark step calls): into a zeroed pool, against what
        # the call that repacks per step writes into a zeroed pool
        dec.expanded_pool.zero_()
        dec.expand_tail(case.d_w_uk, case.d_w_uv, cfg.s_q)
        torch.cuda.synchronize()
        tail_only = dec.expanded_pool.clone()
        assert int((tail_only.view(torch.int16) != 0).sum()) > cfg.B * cfg.s_q * (2 * cfg.g * cfg.d_h) // 2
        dec.pack_expand_weights(case.d_w_uk, case.d_w_uv)
        dec.expanded_pool.zero_()
        dec.expand_tail_packed(cfg.s_q)
        torch.cuda.synchronize()
        assert torch.equal(dec.expanded_pool.view(torch.int16), tail_only.view(torch.int16)), "packed vs unpacked tail expansion"
        del tail_only
        dec.expanded_pool = one_shot
        # 8-bit cache
        dec.alloc_expanded_fp8(fill=0)
        dec.quantize_expanded(1.0, 1.0)
        two_step = dec.expanded_fp8_pool.clone()
        dec.alloc_expanded_fp8(fill=0)
        dec.expand_fp8(case.d_w_uk, case.d_w_uv, 1.0, 1.0)
        torch.cuda.synchronize()
        assert torch.equal(dec.expanded_fp8_pool, two_step), "one-shot 8-bit expansion vs expand + quantise"
        del two_step
        out8, _ = dec.decode_gqa_fp8(case.d(case.q_c), case.d(case.q_r), 1.0, 1.0)
        torch.cuda.synchronize()
        o8 = out8.float().cpu().numpy()
        assert np.isfinite(o8).all()
        for b in (0, 63):
            for j in (1, 6):
                hs = slice(j * G, (j + 1) * G)
                c, kR = case.rows(b)
                KC, V = O.expand_latent(c, case.w_uk[j:j + 1], case.w_uv[j:j + 1])
                kq = F8.dequantize_e4m3(F8.quantize_tensor(S.quantize(KC, cfg.dtype), 1.0))
                vq = F8.dequantize_e4m3(F8.quantize_tensor(S.quantize(V, cfg.dtype), 1.0))
                ref, _ = O.decode_gqa(case.q_c[b][:, hs], case.q_r[b][:, hs], kq, vq, kR)
                check("gqa over the 8-bit cache  b=%d group %d" % (b, j), o8[b][:, hs], ref)
    finally:
        case.close()


def test_c2_absorb_sq1():
    case = FullCase(S.CONFIGS["C2"])
    try:
        q_hat = case.dec.absorb_query(case.d(case.q_c), case.d_w_uk)
        out_a, lse_a = case.dec.decode_absorb(q_hat, case.d(case.q_r), case.d_w_uv)
        torch.cuda.synchronize()
        oa = out_a.float().cpu().numpy()
        assert np.isfinite(oa).all()
        G = 16
        for b in (0, 63):
            for j in (2, 7):
                ref_o, _ = oracle_group(case, b, j, "absorb")
                check("absorb  b=%d group %d" % (b, j), oa[b][:, j * G:(j + 1) * G], ref_o)
    finally:
        case.close()


def test_c2_size_with_the_value_dim_of_the_mla_checkpoints():
    """B = 64, L = 8192 with (d_h, d_v) = (192, 256) (Sec. 3.2.2): the two GPU paths agree with each other on every
    output (Sec. 3.1: one attention output, two routes), and with the oracle on sampled (sequence, group) slices."""
    case = FullCase(S.CONFIGS["C2"].with_(d_h=192, d_v=256, seed=4192))
    try:
        run_both_paths(case, groups_to_check=[0, 5])
    finally:
        case.close()


def test_c2_fp8_latent_at_full_size():
    """The canonical absorb decode over the 8-bit latent cache (Sec. 2 / Sec. 5.1 (i): quantised caches; format of this build): the
    quantising cache switch on the GPU holds the oracle's codes bit for bit on sampled sequences, and the decode is
    checked on sampled (sequence, group) slices against the oracle's MQA-absorb decode (Sec. 3.1) on the dequantised
    latent, consuming the q_hat bits the GPU consumes."""
    from oracle import fp8_cache as F8
    cfg = S.CONFIGS["C2"]
    case = FullCase(cfg)
    dec = case.dec
    c_scale = 2.0 ** -6      # standard-normal latent: |c| / scale stays below 448
    try:
        G = cfg.h_q // cfg.g
        dec.alloc_latent_fp8(fill=0xAA)
        dec.quantize_latent(c_scale)
        q_hat = dec.absorb_query(case.d(case.q_c), case.d_w_uk)
        out8, lse8 = dec.decode_absorb_fp8(q_hat, case.d(case.q_r), c_scale, case.d_w_uv)
        torch.cuda.synchronize()
        o8, l8 = out8.float().cpu().numpy(), lse8.cpu().numpy()
        qh = q_hat.float().cpu().numpy()
        assert np.isfinite(o8).all() and np.isfinite(l8).all()
        pool = dec.latent_fp8_pool.cpu().numpy()
        P, pb = cfg.page_size, F8.latent_fp8_page_bytes(cfg.page_size, cfg.r_kv, cfg.d_r)
        for b in case.sample_sequences(4):
            c, kR = case.rows(b)
            codes = F8.quantize_tensor(c, c_scale)
            # the GPU's codes and k_R bits of this sequence, page by page
            L = int(case.lens[b])
            kr_bits = (np.ascontiguousarray(kR, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
            for p in range((L + P - 1) // P):
                n = min(P, L - p * P)
                base = int(case.table[b][p]) * pb
                assert np.array_equal(pool[base: base + n * cfg.r_kv].reshape(n, cfg.r_kv), codes[p * P: p * P + n]), (b, p)
                got_kr = pool[base + P * cfg.r_kv: base + P * cfg.r_kv + n * cfg.d_r * 2].view(np.uint16).reshape(n, cfg.d_r)
                assert np.array_equal(got_kr, kr_bits[p * P: p * P + n]), (b, p)
            c_deq = F8.dequantize_e4m3(codes) * c_scale
            for j in (0, 3, 7):
                hs = slice(j * G, (j + 1) * G)
                ref_o, ref_l = O.decode_absorb(qh[b][:, hs], case.q_r[b][:, hs], c_deq, kR, case.w_uv[j:j + 1])
                check("absorb over the 8-bit latent  b=%d L=%d group %d" % (b, L, j), o8[b][:, hs], ref_o)
                assert float(np.max(np.abs(l8[b][:, hs] - ref_l))) <= 2e-2
    finally:
        case.close()


def test_c3_single_group_slice():
    """One GPU's share of 8-way head-axis tensor parallelism: group 3 only, 320 cached elements per token."""
    cfg = S.CONFIGS["C3"]
    case = FullCase(cfg, groups=1, group_begin=3)
    try:
        G = cfg.h_q // cfg.g
        hs = slice(3 * G, 4 * G)
        case.dec.alloc_expanded()
        case.dec.expand(case.d_w_uk, case.d_w_uv)
        q_c = np.ascontiguousarray(case.q_c[:, :, hs])
        q_r = np.ascontiguousarray(case.q_r[:, :, hs])
        out, lse = case.dec.decode_gqa(case.d(q_c), case.d(q_r))
        torch.cuda.synchronize()
        og = out.float().cpu().numpy()
        assert np.isfinite(og).all()
        for b in (1, 40):
            ref_o, ref_l = oracle_group(case, b, 3, "gqa")
            check("slice   b=%d group 3" % b, og[b], ref_o)
    finally:
        case.close()


def test_c4_ragged_paged_both_paths():
    case = FullCase(S.CONFIGS["C4"])
    try:
        assert case.lens.min() >= 1024 and case.lens.max() <= 32768
        named = case.named_sequences()
        assert int(np.argmin(case.lens)) in named and int(np.argmax(case.lens)) in named
        assert any(case.lens[b] % cfg_page(case) for b in named), "no sampled length off the page grid"
        # 16 sequences: all 8 groups of the shortest, the longest and one off the page grid; one group (rotating) of the others
        per_seq = run_both_paths(case, groups_to_check=[6], groups_named=range(8), n_seqs=16)
        assert len(per_seq) >= 16
    finally:
        case.close()


def test_c3_compress_rope_and_output_projection_at_full_size():
    """The canonical GQA decode at full size, the shapes bench.py times: the reverse cache switch over all 524288 tokens (sampled
    sequences against the oracle's compression of the oracle's expansion; every recovered latent finite and close to
    the original), the rotary step on all 64 x 2 x 129 vectors (sampled tokens), and W^O with d_model = 7168 on the
    128 rows (four whole rows and 2000 sampled elements against the oracle)."""
    from paper_2605_15250_amd import binding as B
    cfg = S.CONFIGS["C3"]
    case = FullCase(cfg)
    dec = case.dec
    try:
        W = cfg.r_kv + cfg.d_r
        # ---- compress(expand(latent)) ----
        dec.alloc_expanded(fill=0.0)
        dec.expand(case.d_w_uk, case.d_w_uv)
        w_inv = S.quantize(B.gqla_left_inverse(dec.shape, case.w_uk), cfg.dtype)
        truth = dec.latent_pool
        dec.latent_pool = torch.full_like(truth, float("nan"))
        dec.compress(case.d(w_inv))
        torch.cuda.synchronize()
        rec = dec.latent_pool.view(-1, W)
        ref_all = truth.view(-1, W)
        valid = ~torch.isnan(ref_all[:, 0])
        assert bool(torch.isfinite(rec[valid].float()).all())
        assert torch.equal(rec[valid][:, cfg.r_kv:].view(torch.int16), ref_all[valid][:, cfg.r_kv:].view(torch.int16)), "k_R copied bit for bit"
        err = float(torch.linalg.norm(rec[valid][:, :cfg.r_kv].float() - ref_all[valid][:, :cfg.r_kv].float()) /
                    torch.linalg.norm(ref_all[valid][:, :cfg.r_kv].float()))
        print("recovered latent vs the original, all tokens: rel_l2 %.3e" % err, flush=True)
        assert err < 1e-2
        for b in (0, 37):
            c, _ = case.rows(b)
            KC, _ = O.expand_latent(c, case.w_uk, case.w_uv)
            ref = S.quantize(KC, cfg.dtype).reshape(len(c), -1).astype(np.float64) @ w_inv.astype(np.float64).T   # the rounded left inverse the GPU uses
            t = np.arange(int(case.lens[b]))
            slots = torch.from_numpy(case.table[b][t // cfg.page_size].astype(np.int64) * cfg.page_size + t % cfg.page_size).cuda()
            check("compress c_kv  b=%d" % b, rec[slots][:, :cfg.r_kv].float().cpu().numpy(), ref)
        dec.latent_pool = truth
        # ---- rotary step ----
        r = S.rng(cfg.seed, 7)
        rows_raw = S.quantize(r.standard_normal((cfg.B, cfg.s_q, W), dtype=np.float32), cfg.dtype)
        d_q, d_rows = case.d(case.q_r), case.d(rows_raw)
        dec.rope_step(10000.0, d_q, d_rows)
        torch.cuda.synchronize()
        got_q, got_rows = d_q.float().cpu().numpy(), d_rows.float().cpu().numpy()
        assert np.array_equal(got_rows[..., :cfg.r_kv], rows_raw[..., :cfg.r_kv])
        for b in (0, 31, 63):
            for i in range(cfg.s_q):
                t = int(case.lens[b]) - cfg.s_q + i
                check("rope q_R  b=%d tok %d" % (b, i), got_q[b, i], O.rope(case.q_r[b, i], t))
                check("rope k_R  b=%d tok %d" % (b, i), got_rows[b, i, cfg.r_kv:], O.rope(rows_raw[b, i, cfg.r_kv:], t))
        # ---- output projection ----
        d_model = 7168
        w_o = S.output_weights(cfg, d_model)
        o = S.quantize(S.rng(cfg.seed, 8).standard_normal((cfg.B, cfg.s_q, cfg.h_q, cfg.d_h), dtype=np.float32), cfg.dtype)
        y = dec.output_projection(case.d(o), case.d(w_o))
        torch.cuda.synchronize()
        yh = y.float().cpu().numpy().reshape(cfg.B * cfg.s_q, d_model)
        of = o.reshape(cfg.B * cfg.s_q, -1).astype(np.float64)
        assert np.isfinite(yh).all()
        rows4 = [0, 1, 64, 127]
        ref4 = (w_o.astype(np.float64) @ of[rows4].T).T
        for k, m in enumerate(rows4):
            check("W^O row %d" % m, yh[m], ref4[k])
        pick = np.random.default_rng(3).integers(0, [cfg.B * cfg.s_q, d_model], size=(2000, 2))
        ref = np.einsum("ik,ik->i", of[pick[:, 0]], w_o[pick[:, 1]].astype(np.float64))
        check("W^O 2000 sampled elements", yh[pick[:, 0], pick[:, 1]], ref)
    finally:
        case.close()


def test_mla_checkpoint_shape_absorb_path_at_full_size():
    """The absorb path with a value dim of its own at the size bench.py times it (Sec. 3.2.2 shape: h_q = 20, g = 4,
    d_h = 192, d_h^V = 256; B = 64, L = 8192): every output finite, three sequences element by element against the
    oracle (all 20 heads)."""
    cfg = S.CONFIGS["C2"].with_(h_q=20, g=4, d_h=192, d_v=256, B=64, L=8192, s_q=1, seed=15259)
    case = FullCase(cfg)
    try:
        q_hat = case.dec.absorb_query(case.d(case.q_c), case.d_w_uk)
        out, lse = case.dec.decode_absorb(q_hat, case.d(case.q_r), case.d_w_uv)
        torch.cuda.synchronize()
        o, l = out.float().cpu().numpy(), lse.cpu().numpy()
        assert o.shape == (cfg.B, 1, 20, 256) and np.isfinite(o).all() and np.isfinite(l).all()
        for b in (0, 29, 63):
            c, kR = case.rows(b)
            ref_o, ref_l = O.decode_absorb(O.absorb_query(case.q_c[b], case.w_uk), case.q_r[b], c, kR, case.w_uv, d_h=cfg.d_h)
            check("absorb, d_h 192 / d_v 256  b=%d" % b, o[b], ref_o)
            assert float(np.max(np.abs(l[b] - ref_l))) <= 2e-2
    finally:
        case.close()
