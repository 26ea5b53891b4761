#!/usr/bin/env python3
"""Benchmark of the GQLA decode-attention hot path on one MI355X.

One step = one serving step of both decode paths at the paper's canonical shape (h_q=128, g=8, d_h=128, r_kv=512,
d_R=64), B=64 sequences of L=8192 cached tokens, on seeded synthetic data already resident in HBM:
    absorb leg (s_q=1):  gqla_absorb_query -> gqla_decode_absorb   (split-L flash-decode over the latent cache, combine, W_UV)
    GQA leg   (s_q=2):   gqla_append_latent -> gqla_expand_cache_tail_packed -> gqla_decode_gqa
                         (the step's rows into the latent cache, their K_C / V / k_R into the expanded cache from weights
                         repacked once before the steps, grouped decode)
Prints ONE JSON line.  `value` = decoded step tokens per second of that step (B*1 + B*2 tokens per step).  The one-shot
cache switch gqla_expand_cache (Sec. 3.1: done once at deployment) is timed in the same run, outside `value`.
`roofline` is the split-L decode kernel that is further from its target, the absorb decode (kernel time from events
the library records around that kernel inside the timed steps, see gqla_time_next_decode_kernel); `rooflines` has both
decode kernels and the expansion; the per-call times and the GQA kernel's come from passes of the same steps right
behind the timed one (each event is a packet in the stream and would be charged to `value`).  Also in
the line: the other workload shapes (32 heads x 32 sequences with rotating cache buffers so that it is not served from the
last-level cache, 128 ragged sequences, paged), both paths at the operating points of the paper's Sec. 4.2.3 table,
the oracle's CPU rate on a bounded sample, and timings of the calls
around the path (measured ceilings of the chip, the single-group slice, the 8-bit caches, the reverse cache switch, the
rotary step and W^O, each path's whole decode step as one HIP graph, the absorb step with a value dim of its own)."""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X HBM3E
MFMA_BF16_PEAK_TFLOPS = 2500.0
CALIB_COPY_BYTES = 1 << 30
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "hbm_traffic_canonical_bench.txt")   # measured with rocprofv3 --pmc
TRAFFIC_ROWS = {"decode_gqa_bf16_kernel": "decode_gqa", "decode_absorb_shared_bf16_kernel": "decode_absorb", "expand_bf16_kernel": "expand_cache"}


def parse_args():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--batch", type=int, default=0, help="override B (debugging only; changes the workload name)")
    ap.add_argument("--ctx", type=int, default=0, help="override L (debugging only)")
    ap.add_argument("--legs", default="absorb,gqa", help="debugging only: subset of absorb,gqa to run (the judged line needs both)")
    ap.add_argument("--cpu-seqs", type=int, default=64, help="sequences per leg in the oracle's bounded sample (0 = skip)")
    ap.add_argument("--no-extras", action="store_true", help="skip everything outside the timed step (ceiling probes, slice, cache updates, 8-bit cache, compression, step ops)")
    ap.add_argument("--no-operating-points", dest="operating_points", action="store_false",
                    help="skip the operating points of the paper's Sec. 4.2.3 table: both decode paths at (g, s_q) in "
                         "{(8,1), (8,2), (4,1), (4,2)} for B = 1 and 64, L = 8192, timed per call with events")
    ap.add_argument("--crossover", action="store_true",
                    help="also time both decode paths over B = 1 .. 128 (canonical shape, L = 8192, s_q = 1 and 2): where the faster path changes")
    ap.add_argument("--no-other-configs", action="store_true",
                    help="skip the rows of the other workload shapes (32 heads x 32 sequences with rotating cache buffers, 128 sequences, ragged and "
                         "paged; both decode paths and the expansion, five timed calls each, device-generated N(0,1) latents: "
                         "their parity is covered by tests/)")
    return ap.parse_args()


def main():
    args = parse_args()
    if args.gpus != 1:
        print("bench.py: this build measures one GPU only (no sharding or collectives exist in it); run with --gpus 1",
              file=sys.stderr)
        sys.exit(2)
    import torch
    import synth_inputs as S
    from paper_2605_15250_amd import binding as B
    from paper_2605_15250_amd.harness import Decoder, build_latent_pool, to_device

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(2)
    B.lib()  # fails loudly if libgqla.so is missing: there is no fallback path
    torch.cuda.set_device(0)

    legs = {}
    for key, path in (("C2", "absorb"), ("C3", "gqa")):
        cfg = S.CONFIGS[key]
        if args.batch:
            cfg = cfg.with_(B=args.batch)
        if args.ctx:
            cfg = cfg.with_(L=args.ctx)
        lens = S.seq_lens(cfg)
        table, num_pages = S.page_table(cfg, lens)
        dec = Decoder(cfg, lens, table, num_pages, use_page_table=False)   # contiguous cache, identity page map
        dec.latent_pool = build_latent_pool(cfg, lens, table, num_pages, lambda b, L, cfg=cfg: S.sequence_rows(cfg, b, L), fill=0.0)
        w_uk, w_uv = S.weights(cfg)
        q_c, q_r = S.queries(cfg)
        legs[path] = dict(cfg=cfg, lens=lens, table=table, dec=dec, w_uk=w_uk, w_uv=w_uv, q_c=q_c, q_r=q_r,
                          d_w_uk=to_device(w_uk, cfg.dtype), d_w_uv=to_device(w_uv, cfg.dtype),
                          d_q_c=to_device(q_c, cfg.dtype), d_q_r=to_device(q_r, cfg.dtype))
    A, Gq = legs["absorb"], legs["gqa"]
    ca, cg = A["cfg"], Gq["cfg"]
    A["q_hat"] = torch.empty((ca.B, ca.s_q, ca.h_q, ca.r_kv), dtype=torch.bfloat16, device="cuda")
    A["out"] = torch.empty((ca.B, ca.s_q, ca.h_q, ca.d_h), dtype=torch.bfloat16, device="cuda")
    A["lse"] = torch.empty((ca.B, ca.s_q, ca.h_q), dtype=torch.float32, device="cuda")
    Gq["out"] = torch.empty((cg.B, cg.s_q, cg.h_q, cg.d_h), dtype=torch.bfloat16, device="cuda")
    Gq["lse"] = torch.empty((cg.B, cg.s_q, cg.h_q), dtype=torch.float32, device="cuda")
    Gq["dec"].alloc_expanded(fill=0.0)

    names = ["absorb_query", "decode_absorb", "append_latent", "expand_cache_tail", "decode_gqa"]
    kernel_of = {"decode_absorb": "decode_absorb_shared_bf16_kernel", "decode_gqa": "decode_gqa_bf16_kernel"}

    run_legs = set(args.legs.split(","))

    # the GQA leg's step rows: the rows the latent cache already holds at the step's positions, so that the cache
    # content does not change from step to step
    Wl = cg.r_kv + cg.d_r
    pos = torch.stack([torch.from_numpy(Gq["table"][b][(np.arange(int(Gq["lens"][b]) - cg.s_q, int(Gq["lens"][b]))) // cg.page_size].astype(np.int64)
                                        * cg.page_size + (np.arange(int(Gq["lens"][b]) - cg.s_q, int(Gq["lens"][b])) % cg.page_size))
                       for b in range(cg.B)]).cuda()
    step_rows = Gq["dec"].latent_pool.view(-1, Wl)[pos.view(-1)].view(cg.B, cg.s_q, Wl).contiguous()

    def step(events=None, kev_a=None, kev_g=None):
        def rec(i):
            if events is not None:
                events[i].record()
        rec(0)
        if "absorb" in run_legs:
            A["dec"].absorb_query(A["d_q_c"], A["d_w_uk"], A["q_hat"])
        rec(1)
        if "absorb" in run_legs:
            if kev_a is not None:
                B.gqla_time_next_decode_kernel(kev_a[0], kev_a[1])
            A["dec"].decode_absorb(A["q_hat"], A["d_q_r"], A["d_w_uv"], A["out"], A["lse"])
        rec(2)
        if "gqa" in run_legs:
            Gq["dec"].append_latent(step_rows)
        rec(3)
        if "gqa" in run_legs:
            Gq["dec"].expand_tail_packed(cg.s_q)
        rec(4)
        if "gqa" in run_legs:
            if kev_g is not None:
                B.gqla_time_next_decode_kernel(kev_g[0], kev_g[1])
            Gq["dec"].decode_gqa(Gq["d_q_c"], Gq["d_q_r"], Gq["out"], Gq["lse"])
        rec(5)

    # one plain device-to-device copy of known size: the calibration kernel for the HBM traffic counters
    # (FETCH_SIZE / WRITE_SIZE per dispatch are scaled by what they read for this copy)
    calib_src = torch.empty(CALIB_COPY_BYTES, dtype=torch.uint8, device="cuda").fill_(1)
    calib_dst = torch.empty_like(calib_src)
    calib_dst.copy_(calib_src)
    torch.cuda.synchronize()
    del calib_src, calib_dst

    # the one-shot cache switch (deployment time, Sec. 3.1): the GQA leg's expanded cache is complete before the steps
    Gq["dec"].expand(Gq["d_w_uk"], Gq["d_w_uv"])
    # ... and so are the weights in the expansion kernels' operand order: a serving loop repacks them once, not per step
    Gq["dec"].pack_expand_weights(Gq["d_w_uk"], Gq["d_w_uv"])
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(6)] for _ in range(args.steps)]
    kev = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(args.steps)]
    for row in kev:            # torch creates the underlying event on first use: the library needs the handle
        for e in row:
            e.record()
    torch.cuda.synchronize()
    # The timed region carries only the events the top-level roofline needs (the library records them around the absorb
    # decode kernel on this stream).  Every recorded event is a packet of its own in the stream (measured: the six
    # between the calls and the two pairs around the decode kernels took 4 % off `value`), so the per-call breakdown
    # and the second decode kernel's duration come from two more passes of the same steps right behind the timed one.
    t0 = time.perf_counter()
    for k in range(args.steps):
        step(None, kev[k][0:2], None)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_per_step = (t1 - t0) * 1e3 / args.steps
    for k in range(args.steps):
        step(ev[k], None, None)
    torch.cuda.synchronize()
    for k in range(args.steps):
        step(None, None, kev[k][2:4])
    torch.cuda.synchronize()
    call_ms = {n: float(np.mean([ev[k][i].elapsed_time(ev[k][i + 1]) for k in range(args.steps)])) for i, n in enumerate(names)}
    kernel_ms = {}
    if "absorb" in run_legs:
        kernel_ms["decode_absorb"] = float(np.mean([kev[k][0].elapsed_time(kev[k][1]) for k in range(args.steps)]))
    if "gqa" in run_legs:
        kernel_ms["decode_gqa"] = float(np.mean([kev[k][2].elapsed_time(kev[k][3]) for k in range(args.steps)]))

    def timed_steady(fn, reps):
        """Seconds per call over `reps` calls, after at least 40 ms of the same calls: the clock needs some tens of
        milliseconds of load to settle, and the first calls after an idle gap run up to 15 % slower."""
        t0 = time.perf_counter()
        n = 0
        while n < 3 or time.perf_counter() - t0 < 0.04:
            fn()
            n += 1
            if n % 8 == 0:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps * 1e-3

    # ---- the one-shot cache switch, same run, outside `value` ----------------------------------------------------------
    if "gqa" in run_legs:
        call_ms["expand_cache"] = timed_steady(lambda: Gq["dec"].expand(Gq["d_w_uk"], Gq["d_w_uv"]), 5) * 1e3

    # ---- outside the timed step: measured ceilings of this chip, and one rank's share of 8-way head-axis TP ----------
    measured = None
    tp_slice = None
    step_updates = None
    fp8_kv = None
    fp8_latent = None
    compress = None
    step_ops = None
    full_run = run_legs >= {"absorb", "gqa"}
    if full_run and not args.no_extras:
        def timed(fn, reps):
            fn()
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(reps):
                fn()
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / reps * 1e-3
        num_cus = torch.cuda.get_device_properties(0).multi_processor_count
        sink = torch.zeros(4, dtype=torch.int32, device="cuda")
        pool = Gq["dec"].expanded_pool
        unit = 16 * 1024 * 8 * num_cus
        nbytes = pool.numel() * pool.element_size() // unit * unit
        t_rd = timed(lambda: B.gqla_probe_stream_read(pool, nbytes, sink, num_cus), 5)
        iters = 100000
        t_mf = timed(lambda: B.gqla_probe_mfma_bf16(sink, iters, num_cus), 3)
        measured = {"hbm_stream_read_GBs": nbytes / t_rd / 1e9, "mfma_bf16_TFLOPs": B.gqla_probe_mfma_flops(iters, num_cus) / t_mf / 1e12,
                    "how": "gqla_probe_stream_read over %.2f GB (16-byte loads, %d workgroups); gqla_probe_mfma_bf16: register-resident "
                           "32x32x16 bf16 MFMAs with random operand bits, %.0f ms sustained" % (nbytes / 1e9, 8 * num_cus, t_mf * 1e3)}
        # single-group slice of the GQA leg: 16 heads, one group, 320 cached elements per token
        G = cg.h_q // cg.g
        j0 = 3
        sl = Decoder(cg, Gq["lens"], Gq["table"], Gq["dec"].num_pages, groups=1, group_begin=j0, use_page_table=False)
        sl.latent_pool = Gq["dec"].latent_pool
        sl.alloc_expanded(fill=0.0)
        q_c_s = to_device(np.ascontiguousarray(Gq["q_c"][:, :, j0 * G:(j0 + 1) * G]), cg.dtype)
        q_r_s = to_device(np.ascontiguousarray(Gq["q_r"][:, :, j0 * G:(j0 + 1) * G]), cg.dtype)
        out_s = torch.empty((cg.B, cg.s_q, G, cg.d_h), dtype=torch.bfloat16, device="cuda")
        lse_s = torch.empty((cg.B, cg.s_q, G), dtype=torch.float32, device="cuda")
        t_ex = timed(lambda: sl.expand(Gq["d_w_uk"], Gq["d_w_uv"]), 5)
        t_dec = timed(lambda: sl.decode_gqa(q_c_s, q_r_s, out_s, lse_s), 10)
        Lsum = int(Gq["lens"].sum())
        sl_bytes = 2 * Lsum * (2 * cg.d_h + cg.d_r)
        tp_slice = {"groups": 1, "heads": G, "cache_elems_per_token": 2 * cg.d_h + cg.d_r, "decode_gqa_ms": t_dec * 1e3,
                    "GB/s": sl_bytes / t_dec / 1e9, "frac_hbm_peak": sl_bytes / t_dec / 1e9 / HBM_PEAK_GBS,
                    "tokens_per_s": cg.B * cg.s_q / t_dec, "expand_cache_ms": t_ex * 1e3}
        sl.latent_pool = None
        sl.close()
        # the per-step cache updates of the GQA leg: append the step's s_q rows of every sequence and
        # expand just those positions -- what a serving step pays once the context has been expanded in one shot.
        # The rows written are the ones the cache already holds at those positions, so its content does not change.
        gd = Gq["dec"]
        t_app = timed(lambda: gd.append_latent(step_rows), 20)
        t_tail = timed(lambda: gd.expand_tail(Gq["d_w_uk"], Gq["d_w_uv"], cg.s_q), 20)
        t_tail_p = timed(lambda: gd.expand_tail_packed(cg.s_q), 20)
        step_updates = {"append_latent_ms": t_app * 1e3, "expand_cache_tail_ms": t_tail * 1e3,
                        "expand_cache_tail_packed_ms": t_tail_p * 1e3, "tail_tokens": cg.s_q}
        # the GQA leg over an 8-bit expanded cache (K_C, V as E4M3 codes, k_R in 16 bits): 2176 instead of 4224 bytes
        # per token; the quantising cache switch is one-shot, like the expansion
        gd.alloc_expanded_fp8(fill=0)
        t_q = timed(lambda: gd.quantize_expanded(1.0, 1.0), 5)
        two_step = gd.expanded_fp8_pool.clone()
        t_e8 = timed_steady(lambda: gd.expand_fp8(Gq["d_w_uk"], Gq["d_w_uv"], 1.0, 1.0), 5)   # latent -> 8-bit cache in one pass
        same8 = bool(torch.equal(two_step, gd.expanded_fp8_pool))
        del two_step
        out8 = torch.empty_like(Gq["out"])
        t_d8 = timed_steady(lambda: gd.decode_gqa_fp8(Gq["d_q_c"], Gq["d_q_r"], 1.0, 1.0, out8, Gq["lse"]), 20)
        gd.decode_gqa(Gq["d_q_c"], Gq["d_q_r"], Gq["out"], Gq["lse"])
        torch.cuda.synchronize()
        b8 = int(Gq["lens"].sum()) * B.gqla_expanded_fp8_bytes_per_token(cg.g, cg.d_h, cg.d_r)
        d16 = Gq["out"].float()
        fp8_kv = {"quantize_expanded_ms": t_q * 1e3, "expand_cache_fp8_ms": t_e8 * 1e3, "expand_cache_fp8_equals_expand_then_quantize": same8,
                  "decode_gqa_fp8_ms": t_d8 * 1e3, "bytes_per_token": b8 // int(Gq["lens"].sum()),
                  "GB/s": b8 / t_d8 / 1e9, "frac_hbm_peak": b8 / t_d8 / 1e9 / HBM_PEAK_GBS, "tokens_per_s": cg.B * cg.s_q / t_d8,
                  "rel_l2_vs_16bit_cache": float(torch.linalg.norm(out8.float() - d16) / torch.linalg.norm(d16))}
        gd.expanded_fp8_pool = None
        del out8
        # the absorb leg (128 heads) over an 8-bit latent cache (c_kv as E4M3 codes with one scale, k_R in 16 bits):
        # 640 instead of 1152 bytes per token.  The scale 2^-6 keeps the standard-normal latent of this workload inside
        # the format's range.  Decode kernel timed by the library's events, as for the 16-bit cache.
        ad = A["dec"]
        c8 = 2.0 ** -6
        ad.alloc_latent_fp8(fill=0)
        t_ql = timed(lambda: ad.quantize_latent(c8), 5)
        outl8 = torch.empty_like(A["out"])
        lat8_call = lambda: ad.decode_absorb_fp8(A["q_hat"], A["d_q_r"], c8, A["d_w_uv"], outl8, A["lse"])
        t_l8 = timed_steady(lat8_call, 20)
        pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(10)]
        for e0, e1 in pairs:
            e0.record()
            e1.record()
        for e0, e1 in pairs:
            B.gqla_time_next_decode_kernel(e0, e1)
            lat8_call()
        torch.cuda.synchronize()
        k_l8 = float(np.mean([e0.elapsed_time(e1) for e0, e1 in pairs])) * 1e-3
        ad.decode_absorb(A["q_hat"], A["d_q_r"], A["d_w_uv"], A["out"], A["lse"])
        torch.cuda.synchronize()
        La_ = int(A["lens"].sum())
        bl8 = La_ * B.gqla_latent_fp8_bytes_per_token(ca.r_kv, ca.d_r)
        fl8 = 2.0 * La_ * ca.h_q * ca.s_q * (2 * ca.r_kv + ca.d_r)
        a16 = A["out"].float()
        fp8_latent = {"quantize_latent_ms": t_ql * 1e3, "decode_absorb_fp8_ms": t_l8 * 1e3, "kernel": "decode_absorb_shared_bf16_kernel",
                      "kernel_ms": k_l8 * 1e3, "bytes_per_token": bl8 // La_, "c_scale": c8,
                      "GB/s": bl8 / k_l8 / 1e9, "frac_hbm_peak": bl8 / k_l8 / 1e9 / HBM_PEAK_GBS,
                      "TFLOP/s": fl8 / k_l8 / 1e12, "frac_mfma_peak": fl8 / k_l8 / 1e12 / MFMA_BF16_PEAK_TFLOPS,
                      "tokens_per_s": ca.B * ca.s_q / t_l8,
                      "rel_l2_vs_16bit_cache": float(torch.linalg.norm(outl8.float() - a16) / torch.linalg.norm(a16))}
        ad.latent_fp8_pool = None
        del outl8, a16
        # the reverse cache switch (expanded -> latent through the left inverse of the stacked key up-projection)
        import time as _time
        t0 = _time.perf_counter()
        w_inv = B.gqla_left_inverse(gd.shape, Gq["w_uk"])
        t_inv = _time.perf_counter() - t0
        d_w_inv = to_device(S.quantize(w_inv, cg.dtype), cg.dtype)
        truth = gd.latent_pool
        gd.latent_pool = torch.zeros_like(truth)
        t_cmp = timed_steady(lambda: gd.compress(d_w_inv), 10)
        rec = gd.latent_pool.view(-1, Wl)[pos.view(-1)][:, :cg.r_kv].float()
        ref = truth.view(-1, Wl)[pos.view(-1)][:, :cg.r_kv].float()
        cmp_flops = 2.0 * Lsum * cg.g * cg.d_h * cg.r_kv
        compress = {"left_inverse_host_ms": t_inv * 1e3, "compress_cache_ms": t_cmp * 1e3, "TFLOP/s": cmp_flops / t_cmp / 1e12,
                    "frac_mfma_peak": cmp_flops / t_cmp / 1e12 / MFMA_BF16_PEAK_TFLOPS,
                    "rel_l2_recovered_latent": float(torch.linalg.norm(rec - ref) / torch.linalg.norm(ref))}
        gd.latent_pool = truth
        del rec, ref, d_w_inv
        # the steps either side of the path: rotary embedding of the step's q_R / k_R and the output projection W^O
        # (d_model 4096 with 32 heads, 7168 with 128: the model widths the two head counts come from)
        step_ops = {}
        for nm, leg in (("absorb", A), ("gqa", Gq)):
            c_, d_ = leg["cfg"], leg["dec"]
            d_model = 4096 if c_.h_q * c_.d_h <= 4096 else 7168
            w_o = to_device(S.output_weights(c_, d_model), c_.dtype)
            y = torch.empty((c_.B, c_.s_q, d_model), dtype=torch.bfloat16, device="cuda")
            o_in = leg["out"]
            # three weight matrices in turn, as the layers of a model would bring them: one matrix alone (235 MB at 128
            # heads) would be served in part by the 256 MB last-level cache from one timed call to the next
            w_turn = [w_o, torch.roll(w_o, 1, 0), torch.roll(w_o, 2, 0)]
            turn = [0]

            def out_proj_call():
                turn[0] = (turn[0] + 1) % 3
                d_.output_projection(o_in, w_turn[turn[0]], y)
            t_o = timed_steady(out_proj_call, 21)
            del w_turn
            q_tmp = leg["d_q_r"].clone()
            rows_tmp = torch.zeros((c_.B, c_.s_q, c_.r_kv + c_.d_r), dtype=torch.bfloat16, device="cuda")
            t_r = timed_steady(lambda: d_.rope_step(10000.0, q_tmp, rows_tmp), 20)
            wbytes = 2.0 * d_model * c_.h_q * c_.d_h
            step_ops[nm] = {"d_model": d_model, "rows": c_.B * c_.s_q, "output_projection_ms": t_o * 1e3,
                            "output_projection_GB/s": wbytes / t_o / 1e9, "frac_hbm_peak": wbytes / t_o / 1e9 / HBM_PEAK_GBS,
                            "rope_step_ms": t_r * 1e3}
            # the whole decode step of this path as one HIP graph: rope -> append -> (absorb: query absorption + latent
            # decode | GQA: tail expansion + grouped decode) -> W^O.  The step's rows are the ones the cache already
            # holds at those positions (their k_R gets rotated by the replays; restored below).
            Wl_ = c_.r_kv + c_.d_r
            lens_ = leg["lens"]
            pos_ = torch.stack([torch.from_numpy(leg["table"][b][np.arange(int(lens_[b]) - c_.s_q, int(lens_[b])) // c_.page_size].astype(np.int64)
                                                 * c_.page_size + np.arange(int(lens_[b]) - c_.s_q, int(lens_[b])) % c_.page_size)
                                for b in range(c_.B)]).cuda()
            rows0 = d_.latent_pool.view(-1, Wl_)[pos_.view(-1)].view(c_.B, c_.s_q, Wl_).contiguous()
            rows_t, q_r_t = rows0.clone(), leg["d_q_r"].clone()
            out_t, lse_t = torch.empty_like(leg["out"]), torch.empty_like(leg["lse"])

            def whole_step():
                d_.rope_step(10000.0, q_r_t, rows_t)
                d_.append_latent(rows_t)
                if nm == "absorb":
                    d_.absorb_query(leg["d_q_c"], leg["d_w_uk"], leg["q_hat"])
                    d_.decode_absorb(leg["q_hat"], q_r_t, leg["d_w_uv"], out_t, lse_t)
                else:
                    d_.expand_tail_packed(c_.s_q)
                    d_.decode_gqa(leg["d_q_c"], q_r_t, out_t, lse_t)
                d_.output_projection(out_t, w_o, y)

            whole_step()
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                whole_step()
            t_s = timed_steady(graph.replay, 20)
            step_ops[nm].update({"whole_step_graph_ms": t_s * 1e3, "whole_step_tokens_per_s": c_.B * c_.s_q / t_s})
            d_.append_latent(rows0)                              # put the cache back as it was
            if nm == "gqa":
                d_.expand_tail(leg["d_w_uk"], leg["d_w_uv"], c_.s_q)
            torch.cuda.synchronize()
            del graph, w_o, y, q_tmp, rows_tmp, rows_t, q_r_t, out_t, lse_t

    # the absorb path with a value dim of its own (Sec. 3.2.2: the MLA checkpoint shape h_q = 20, d_h = 192, d_h^V = 256,
    # r_kv = 512, here with g = 4): B = 64 sequences of 8192 tokens, device-generated latents (timing only; parity of
    # the shape is in the tests)
    mla_shape = None
    if full_run and not args.no_extras:
        c = S.CONFIGS["C2"].with_(h_q=20, g=4, d_h=192, d_v=256, B=64, L=8192, s_q=1)
        lens_k = S.seq_lens(c)
        table_k, np_k = S.page_table(c, lens_k)
        dk = Decoder(c, lens_k, table_k, np_k, use_page_table=False)
        dk.latent_pool = torch.empty(np_k * c.page_size * (c.r_kv + c.d_r), dtype=torch.bfloat16, device="cuda").normal_()
        wk, wv = S.weights(c)
        qc_k, qr_k = S.queries(c)
        d_wk, d_wv, d_qc, d_qr = (to_device(x, c.dtype) for x in (wk, wv, qc_k, qr_k))
        o_k = torch.empty((c.B, c.s_q, c.h_q, c.dv), dtype=torch.bfloat16, device="cuda")
        l_k = torch.empty((c.B, c.s_q, c.h_q), dtype=torch.float32, device="cuda")
        qh_k = torch.empty((c.B, c.s_q, c.h_q, c.r_kv), dtype=torch.bfloat16, device="cuda")

        def mla_step():
            dk.absorb_query(d_qc, d_wk, qh_k)
            dk.decode_absorb(qh_k, d_qr, d_wv, o_k, l_k)
        t_m = timed_steady(mla_step, 20)
        b_m = 2 * int(lens_k.sum()) * (c.r_kv + c.d_r)
        mla_shape = {"h_q": c.h_q, "g": c.g, "d_h": c.d_h, "d_v": c.dv, "batch": c.B, "context": c.L, "absorb_step_ms": t_m * 1e3,
                     "GB/s": b_m / t_m / 1e9, "frac_hbm_peak": b_m / t_m / 1e9 / HBM_PEAK_GBS, "tokens_per_s": c.B * c.s_q / t_m,
                     "finite": bool(torch.isfinite(o_k.float()).all())}
        dk.close()
        del dk, o_k, l_k, qh_k

    # ---- the other workload shapes: LLaMA-3-8B-converted (h_q = 32) and 128 sequences (ragged, paged, s_q = 2) ----
    # Five timed calls each after a short steady warm-up.  The first one's latent cache (151 MB) would fit the chip's 256 MB
    # last-level cache if the same buffer were decoded again and again, so four copies of it are decoded in rotation
    # (604 MB between two uses of a line); the other caches are larger than that cache to begin with.
    other = None
    if full_run and not args.no_other_configs:
        other = []
        for key in ("C1", "C4"):
            c = S.CONFIGS[key]
            lens_k = S.seq_lens(c)
            table_k, np_k = S.page_table(c, lens_k)
            dk = Decoder(c, lens_k, table_k, np_k, use_page_table=c.paged)
            n_elems = np_k * c.page_size * (c.r_kv + c.d_r)
            n_rot = 4 if 2 * n_elems < (1 << 28) else 1
            pools = [torch.empty(n_elems, dtype=torch.bfloat16, device="cuda").normal_() for _ in range(n_rot)]
            dk.latent_pool = pools[0]
            wk, wv = S.weights(c)
            qc_k, qr_k = S.queries(c)
            d_wk, d_wv, d_qc, d_qr = (to_device(x, c.dtype) for x in (wk, wv, qc_k, qr_k))
            o_k = torch.empty((c.B, c.s_q, c.h_q, c.d_h), dtype=torch.bfloat16, device="cuda")
            l_k = torch.empty((c.B, c.s_q, c.h_q), dtype=torch.float32, device="cuda")
            qh_k = dk.absorb_query(d_qc, d_wk)
            turn = [0]

            def absorb_call():
                turn[0] += 1
                dk.latent_pool = pools[turn[0] % n_rot]
                dk.decode_absorb(qh_k, d_qr, d_wv, o_k, l_k)

            def kernel_time(call, reps=5):
                """mean time of the split-L decode kernel inside `call` (events recorded by the library)"""
                pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(reps)]
                for e0, e1 in pairs:
                    e0.record()
                    e1.record()
                for e0, e1 in pairs:
                    B.gqla_time_next_decode_kernel(e0, e1)
                    call()
                torch.cuda.synchronize()
                return float(np.mean([e0.elapsed_time(e1) for e0, e1 in pairs])) * 1e-3
            t_a = timed_steady(absorb_call, 5)
            k_a = kernel_time(absorb_call)
            dk.latent_pool = pools[0]
            dk.alloc_expanded(fill=0.0)
            t_e = timed_steady(lambda: dk.expand(d_wk, d_wv), 5)
            gqa_call = lambda: dk.decode_gqa(d_qc, d_qr, o_k, l_k)
            t_g = timed_steady(gqa_call, 5)
            k_g = kernel_time(gqa_call)
            Ls = int(lens_k.sum())
            b_a, f_a = 2 * Ls * (c.r_kv + c.d_r), 2 * Ls * c.h_q * c.s_q * (2 * c.r_kv + c.d_r)
            b_g, f_e = 2 * Ls * (2 * c.g * c.d_h + c.d_r), 2 * Ls * c.r_kv * 2 * c.g * c.d_h
            other.append({"config": key, "batch": c.B, "h_q": c.h_q, "s_q": c.s_q, "cached_tokens": Ls, "paged": bool(c.paged),
                          "latent_buffers_in_rotation": n_rot, "timed_calls": 5,
                          "decode_absorb": {"ms": t_a * 1e3, "kernel_ms": k_a * 1e3, "tokens_per_s": c.B * c.s_q / t_a,
                                            "GB/s": b_a / t_a / 1e9, "TFLOP/s": f_a / t_a / 1e12,
                                            "frac_hbm_peak": b_a / t_a / 1e9 / HBM_PEAK_GBS, "frac_mfma_peak": f_a / t_a / 1e12 / MFMA_BF16_PEAK_TFLOPS,
                                            "kernel_frac_hbm_peak": b_a / k_a / 1e9 / HBM_PEAK_GBS,
                                            "kernel_frac_mfma_peak": f_a / k_a / 1e12 / MFMA_BF16_PEAK_TFLOPS},
                          "decode_gqa": {"ms": t_g * 1e3, "kernel_ms": k_g * 1e3, "tokens_per_s": c.B * c.s_q / t_g,
                                         "GB/s": b_g / t_g / 1e9, "frac_hbm_peak": b_g / t_g / 1e9 / HBM_PEAK_GBS,
                                         "kernel_frac_hbm_peak": b_g / k_g / 1e9 / HBM_PEAK_GBS},
                          "expand_cache": {"ms": t_e * 1e3, "TFLOP/s": f_e / t_e / 1e12, "frac_mfma_peak": f_e / t_e / 1e12 / MFMA_BF16_PEAK_TFLOPS}})
            dk.close()
            del dk, o_k, l_k, qh_k, pools
            torch.cuda.empty_cache()

    # ---- the operating points of the paper's table (Sec. 4.2.3: L = 8192, absorb vs GQA at (g, s_q)), measured ----------
    # Calls are timed with events (absorb: query absorption + decode; GQA: decode only, the expansion is one-shot at
    # deployment), the model columns are the paper's max(F/peak, B/BW) with this run's measured ceilings.
    points = None
    crossover = None
    if args.operating_points or args.crossover:
        timed3 = timed_steady
        rates = (measured["hbm_stream_read_GBs"] * 1e9, measured["mfma_bf16_TFLOPs"] * 1e12) if measured else (HBM_PEAK_GBS * 1e9, MFMA_BF16_PEAK_TFLOPS * 1e12)
        points = [] if args.operating_points else None
        crossover = [] if args.crossover else None
        todo = []
        if args.operating_points:       # the paper's table (Sec. 4.2.3), at B = 1 and 64
            todo += [(points, Bn, 128, g_k, sq_k) for Bn in (1, 64) for g_k, sq_k in ((8, 1), (8, 2), (4, 1), (4, 2))]
            todo += [(points, 64, 64, 8, sq_k) for sq_k in (1, 2)]     # h_q = 64 (Sec. 4.2: recent open models; every intensity halves)
        if args.crossover:              # where the faster path changes with the batch, canonical shape
            todo += [(crossover, Bn, 128, 8, sq_k) for sq_k in (1, 2) for Bn in (1, 2, 4, 8, 16, 32, 64, 128)]
        for sink_list, Bn, hq_k, g_k, sq_k in todo:
            c = S.CONFIGS["C2"].with_(B=Bn, h_q=hq_k, g=g_k, s_q=sq_k)
            lens_k = S.seq_lens(c)
            table_k, np_k = S.page_table(c, lens_k)
            dk = Decoder(c, lens_k, table_k, np_k, use_page_table=False)
            dk.latent_pool = torch.empty(np_k * c.page_size * (c.r_kv + c.d_r), dtype=torch.bfloat16, device="cuda").normal_()
            wk, wv = S.weights(c)
            qc_k, qr_k = S.queries(c)
            d_wk, d_wv, d_qc, d_qr = (to_device(x, c.dtype) for x in (wk, wv, qc_k, qr_k))
            o_k = torch.empty((c.B, c.s_q, c.h_q, c.d_h), dtype=torch.bfloat16, device="cuda")
            l_k = torch.empty((c.B, c.s_q, c.h_q), dtype=torch.float32, device="cuda")
            qh_k = torch.empty((c.B, c.s_q, c.h_q, c.r_kv), dtype=torch.bfloat16, device="cuda")

            def absorb_step():
                dk.absorb_query(d_qc, d_wk, qh_k)
                dk.decode_absorb(qh_k, d_qr, d_wv, o_k, l_k)
            t_a = timed3(absorb_step, 20)
            dk.alloc_expanded(fill=0.0)
            dk.expanded_pool.normal_()
            t_g = timed3(lambda: dk.decode_gqa(d_qc, d_qr, o_k, l_k), 20)
            Ls = int(lens_k.sum())
            est = B.gqla_estimate_paths(B.make_shape(c.B, c.h_q, c.g, c.d_h, c.r_kv, c.d_r, c.s_q, B.GQLA_BF16), Ls, rates[0], rates[1])
            sink_list.append({"batch": Bn, "context": c.L, "h_q": hq_k, "g": g_k, "s_q": sq_k,
                           "absorb_bytes_per_token": 2 * (c.r_kv + c.d_r), "gqa_bytes_per_token": 2 * (2 * c.g * c.d_h + c.d_r),
                           "absorb_intensity": est["absorb_intensity"], "gqa_intensity": est["gqa_intensity"],
                           "absorb_us": t_a * 1e6, "gqa_us": t_g * 1e6,
                           "absorb_tokens_per_s": Bn * sq_k / t_a, "gqa_tokens_per_s": Bn * sq_k / t_g,
                           "faster_path": "gqa" if t_g < t_a else "absorb",
                           "model_absorb_us": est["absorb_seconds"] * 1e6, "model_gqa_us": est["gqa_seconds"] * 1e6,
                           "model_faster_path": "gqa" if est["faster_path"] == B.GQLA_PATH_GQA else "absorb",
                           "calibrated": (lambda ch: {"absorb_us": ch["absorb_seconds"] * 1e6, "gqa_us": ch["gqa_seconds"] * 1e6,
                                                      "path": "gqa" if ch["faster_path"] == B.GQLA_PATH_GQA else "absorb"})(
                               B.gqla_select_path(B.make_shape(c.B, c.h_q, c.g, c.d_h, c.r_kv, c.d_r, c.s_q, B.GQLA_BF16), Ls))})
            dk.close()
            del dk, o_k, l_k, qh_k
            torch.cuda.empty_cache()

    # ---- accounting: the paper's closed forms (Sec. 4.2.1 / 4.2.2) ----------------------------------------------
    La, Lg = int(A["lens"].sum()), int(Gq["lens"].sum())
    bytes_absorb = 2 * La * (ca.r_kv + ca.d_r)
    flops_absorb = 2 * La * ca.h_q * ca.s_q * (2 * ca.r_kv + ca.d_r)
    bytes_gqa = 2 * Lg * (2 * cg.g * cg.d_h + cg.d_r)
    flops_gqa = 2 * Lg * cg.h_q * cg.s_q * (2 * cg.d_h + cg.d_r)
    bytes_expand = bytes_gqa + 2 * Lg * (cg.r_kv + cg.d_r)
    flops_expand = 2 * Lg * cg.r_kv * 2 * cg.g * cg.d_h

    traffic = {}
    if os.path.exists(TRAFFIC_FILE) and not args.batch and not args.ctx:
        # rows of the committed summary: kernel, FETCH_SIZE, read MB, WRITE_SIZE, written MB, read/alg
        with open(TRAFFIC_FILE) as fh:
            for ln in fh:
                f = ln.split()
                if len(f) == 6 and f[0] in TRAFFIC_ROWS:
                    traffic[TRAFFIC_ROWS[f[0]]] = int(round((float(f[2]) + float(f[4])) * 1e6))

    TARGET = {"decode_absorb": 0.60, "decode_gqa": 0.70}   # of the MFMA peak / of the HBM peak

    def roof(name, bound, nbytes, flops):
        # decode calls: the split-L decode KERNEL (events recorded by the library around it); expansion: the call
        t_ms = kernel_ms.get(name, call_ms[name])
        t = max(t_ms, 1e-6) * 1e-3
        gbs, tf = nbytes / t / 1e9, flops / t / 1e12
        intensity = flops / nbytes
        attainable_tf = min(intensity * HBM_PEAK_GBS / 1e3, MFMA_BF16_PEAK_TFLOPS)
        r = {"call": name, "kernel": kernel_of.get(name, "expand_bf16_kernel (+ pack_weights_bf16_kernel, one call)"),
             "timed": "kernel" if name in kernel_ms else "call", "ms": t_ms, "call_ms": call_ms[name],
             "GB/s": gbs, "TFLOP/s": tf, "frac_hbm_peak": gbs / HBM_PEAK_GBS,
             "frac_mfma_peak": tf / MFMA_BF16_PEAK_TFLOPS, "frac_of_min_roof": tf / attainable_tf,
             "algorithmic_bytes": nbytes, "algorithmic_flops": flops}
        if bound == "hbm":
            r.update({"bound": "hbm", "achieved": gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": gbs / HBM_PEAK_GBS})
        else:
            r.update({"bound": "mfma", "achieved": tf, "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                      "frac": tf / MFMA_BF16_PEAK_TFLOPS})
        if name in TARGET:
            r["target_frac"] = TARGET[name]
        r["traffic"] = traffic.get(name)
        if measured:
            r["frac_of_measured"] = {"hbm_stream_read": gbs / measured["hbm_stream_read_GBs"], "mfma_bf16": tf / measured["mfma_bf16_TFLOPs"]}
        return r

    roofs = []
    if "absorb" in run_legs:
        roofs.append(roof("decode_absorb", "mfma", bytes_absorb, flops_absorb))
    if "gqa" in run_legs:
        roofs.append(roof("decode_gqa", "hbm", bytes_gqa, flops_gqa))
        roofs.append(roof("expand_cache", "mfma", bytes_expand, flops_expand))
    # the line's roofline: of the two decode kernels the metric names, the one further from its target
    dominant = min((r for r in roofs if "target_frac" in r), key=lambda r: r["frac"] / r["target_frac"])
    tokens_per_step = (ca.B * ca.s_q if "absorb" in run_legs else 0) + (cg.B * cg.s_q if "gqa" in run_legs else 0)
    value = tokens_per_step / (ms_per_step * 1e-3)

    # ---- the oracle on a bounded sample of the same workload, and a parity spot check ---------------------------------
    cpu = None
    parity = None
    if args.cpu_seqs > 0:
        from oracle import gqla_oracle as O
        try:
            from threadpoolctl import threadpool_info
            cores = max([p.get("num_threads", 1) for p in threadpool_info()] + [1])
        except Exception:
            cores = len(os.sched_getaffinity(0))
        nb = min(args.cpu_seqs, ca.B)
        out_a = A["out"].float().cpu().numpy()
        out_g = Gq["out"].float().cpu().numpy()
        ref_a, ref_g = [], []
        rows_a = [S.sequence_rows(ca, b, A["lens"][b]) for b in range(nb)]
        rows_g = [S.sequence_rows(cg, b, Gq["lens"][b]) for b in range(nb)]
        t_cpu = t_exp = 0.0
        for b in range(nb):
            c, kR = rows_a[b][:, :ca.r_kv], rows_a[b][:, ca.r_kv:]
            tc0 = time.perf_counter()
            qh = O.absorb_query(A["q_c"][b], A["w_uk"])
            ref_a.append(O.decode_absorb(qh, A["q_r"][b], c, kR, A["w_uv"])[0])
            t_cpu += time.perf_counter() - tc0
            c, kR = rows_g[b][:, :cg.r_kv], rows_g[b][:, cg.r_kv:]
            tc0 = time.perf_counter()
            KC, V = O.expand_latent(c, Gq["w_uk"], Gq["w_uv"])     # the one-shot cache switch: outside the step on both sides
            t_exp += time.perf_counter() - tc0
            tc0 = time.perf_counter()
            ref_g.append(O.decode_gqa(Gq["q_c"][b], Gq["q_r"][b], KC, V, kR)[0])
            t_cpu += time.perf_counter() - tc0
        cpu = {"value": nb * (ca.s_q + cg.s_q) / t_cpu, "unit": "tokens/s", "cores": int(cores), "kind": "oracle",
               "sample": "first %d of %d sequences of each leg at L=%d: absorb_query + decode_absorb (s_q=1) and decode_gqa on the "
                         "oracle's expansion (s_q=2), numpy fp64 (BLAS-backed matmuls, not plain loops), %.1f s; the expansion "
                         "itself, one-shot on both sides, took the oracle another %.1f s" % (nb, ca.B, ca.L, t_cpu, t_exp)}
        ref_a, ref_g = np.stack(ref_a), np.stack(ref_g)

        def errs(got, ref):
            per_seq = [float(np.linalg.norm(got[b] - ref[b]) / np.linalg.norm(ref[b])) for b in range(len(ref))]
            return {"max_abs": float(np.max(np.abs(got - ref))), "rel_l2": float(np.linalg.norm(got - ref) / np.linalg.norm(ref)),
                    "rel_l2_per_sequence_max": max(per_seq), "rel_l2_per_sequence_median": float(np.median(per_seq))}
        parity = {"absorb_vs_oracle": errs(out_a[:nb], ref_a), "gqa_vs_oracle": errs(out_g[:nb], ref_g),
                  "tolerance": {"max_abs": 2e-2, "rel_l2": 1e-2}}

    # ---- the paper's path-selection model (Sec. 4.2.3) evaluated with this chip's measured ceilings --------------------
    path_model = None
    if measured:
        path_model = {"rates": "measured_peaks (this run)"}
        for leg, c, Ltot in (("absorb_leg_s_q1", ca, La), ("gqa_leg_s_q2", cg, Lg)):
            est = B.gqla_estimate_paths(B.make_shape(c.B, c.h_q, c.g, c.d_h, c.r_kv, c.d_r, c.s_q, B.GQLA_BF16), Ltot,
                                        measured["hbm_stream_read_GBs"] * 1e9, measured["mfma_bf16_TFLOPs"] * 1e12)
            path_model[leg] = {"model_absorb_us": est["absorb_seconds"] * 1e6, "model_gqa_us": est["gqa_seconds"] * 1e6,
                               "model_faster_path": "gqa" if est["faster_path"] == B.GQLA_PATH_GQA else "absorb",
                               "ridge": est["ridge"], "absorb_intensity": est["absorb_intensity"], "gqa_intensity": est["gqa_intensity"]}
        path_model["absorb_leg_s_q1"]["measured_absorb_us"] = call_ms["decode_absorb"] * 1e3
        path_model["gqa_leg_s_q2"]["measured_gqa_us"] = call_ms["decode_gqa"] * 1e3

    wl = ("canonical (h_q=128,g=8,d_h=128,r_kv=512,d_R=64) B=%d L=%d: configs[2] absorb decode s_q=1 + configs[3] GQA decode s_q=2 "
          "(append + tail expansion from weights repacked once + decode; the one-shot expansion is timed beside the step, in calls_ms and rooflines)" % (ca.B, ca.L))
    line = {
        "metric": "decode attn tokens/s + % roofline (MFMA absorb, HBM GB/s GQA) on 1 MI355X",
        "value": value, "unit": "tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": wl, "batch": ca.B, "context": ca.L, "tokens_per_step": tokens_per_step,
                   "page_size": ca.page_size, "cache": "contiguous"},
        "roofline": {k: dominant[k] for k in ("bound", "achieved", "peak", "unit", "frac", "traffic", "kernel", "target_frac")}
                    | {"kernel_us": dominant["ms"] * 1e3},
        "rooflines": roofs,
        "measured_peaks": measured,
        "path_model": path_model,
        "tp_slice": tp_slice,
        "step_updates": step_updates,
        "fp8_kv": fp8_kv,
        "fp8_latent": fp8_latent,
        "compress": compress,
        "step_ops": step_ops,
        "mla_shape": mla_shape,
        "other_configs": other,
        "operating_points": points,
        "crossover": crossover,
        "calls_ms": call_ms,
        "kernels_ms": kernel_ms,
        "paths": {"absorb_tokens_per_s": ca.B * ca.s_q / (max(call_ms["absorb_query"] + call_ms["decode_absorb"], 1e-6) * 1e-3),
                  "gqa_decode_tokens_per_s": cg.B * cg.s_q / (max(call_ms["decode_gqa"], 1e-6) * 1e-3),
                  "gqa_step_tokens_per_s": cg.B * cg.s_q / (max(call_ms["append_latent"] + call_ms["expand_cache_tail"] + call_ms["decode_gqa"], 1e-6) * 1e-3),
                  "gqa_step_with_full_expansion_tokens_per_s": (cg.B * cg.s_q / ((call_ms["expand_cache"] + call_ms["decode_gqa"]) * 1e-3))
                  if "expand_cache" in call_ms else None},
        "cpu_baseline": cpu,
        "parity": parity,
    }
    print(json.dumps(line))
    for leg in legs.values():
        leg["dec"].close()


if __name__ == "__main__":
    main()
