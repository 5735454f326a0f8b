#!/usr/bin/env python3
"""Benchmark of the Aggressive Decoding hot path on one MI355X.

Workload of the headline number: Transformer-base input-guided decoding at batch 1 (6+6
layers, d 512, 8 heads, FFN 2048, vocab 32000, bf16 weights, fp32 accumulation), source
lengths ~ N(25, 8) clipped to [5, 64], output length = source length, guide = the model's
greedy output with i.i.d. edits at rate 0.1.  One step = one whole decode of one sentence:
encoder forward + cross-attention keys/values, then the draft-verify loop (row assembly,
verify forward with fused output projection / arg max, prefix match, accept, rollback)
until the output is complete.  Value = emitted tokens per second over the timed steps; every
emitted sequence is checked to be identical to greedy decoding on the same kernels.

Also reported in the same JSON line: `roofline`, the verify forward at batch 1 against the HBM
roofline (its algorithmic bytes over its measured duration), `roofline_bs32`, the verify forward
at batch 32 (first-iteration shape) against the bf16 MFMA roofline, the figures of the largest
single kernel (output projection + arg max) under `vocab_kernel`, and the CPU oracle timed on
this machine's host cores on a bounded sample.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK = 8.0e12       # B/s, MI355X published
MFMA_BF16_PEAK = 2.5e15  # FLOP/s dense bf16, MI355X published


# HBM bytes per launch of the output-projection kernel at the headline shape (base model, 17..32
# rows), from two rocprofv3 --pmc runs of this file (FETCH_SIZE 16336.9 KiB x 2.000, WRITE_SIZE
# 482.7 KiB x 1.0; factors from k_calibration_copy's readings for a 256 MiB copy in the same runs;
# profiles/bench_base_bs1_vocab_kernel_hbm_traffic.md): a figure of an earlier counter run, quoted
# under `vocab_kernel.traffic_from_profile`, not a reading of this run
VOCAB_KERNEL_TRAFFIC_BYTES = int(16336.9 * 1024 * (262144.0 / 131083.0) + 482.7 * 1024)
# HBM bytes of one verify forward of the base model at batch 1, 25 rows, with a launch per stage (no counter run
# exists of the one whose layers are one launch): the sum over its 45 launches of
# FETCH_SIZE (48909.7 KiB x 2.000) and WRITE_SIZE (3566.1 KiB x 1.000) per dispatch, two rocprofv3 --pmc
# runs of `bench.py --profile-forward 1 25 --calibration-copy`
# (profiles/verify_forward_base_bs1_25rows_hbm_traffic.md).  A figure of that counter run, not a reading
# of this one; the row count of the forward timed below may differ by a few rows, which moves it by
# well under 1 % (weights are 98 % of it).
VERIFY_FORWARD_TRAFFIC_BYTES = int(48909.7 * 1024 * (262144.0 / 131084.9) + 3566.1 * 1024)


def decoder_stream_params(dims):
    """Parameters a verify forward streams: per decoder layer self-attn 4d^2, cross-attn q,o 2d^2,
    FFN 2dF; plus the output projection dV."""
    d, F, V, NL = dims["d_model"], dims["d_ffn"], dims["vocab"], dims["dec_layers"]
    return NL * (6 * d * d + 2 * d * F) + d * V


def _progress(what):
    """One line per section on stderr: a long run shows that it is alive; stdout carries the JSON line alone."""
    print(f"bench.py: {what}", file=sys.stderr, flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=256)
    ap.add_argument("--warmup", type=int, default=64)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-bs32", action="store_true")
    ap.add_argument("--no-gad", action="store_true", help="skip the block-drafter workloads 3 and 4")
    ap.add_argument("--no-graphs", action="store_true", help="launch every kernel eagerly (AD_OPT_GRAPHS = 0)")
    ap.add_argument("--no-next", action="store_true", help="skip the row/batch sweeps and the deep-encoder workload")
    ap.add_argument("--cpu-sentences", type=int, default=256)
    ap.add_argument("--sentences", type=int, default=0,
                    help="use only the first N sentences of the batch-1 workload (counter runs, where every "
                         "launch is serialised); 0 = all")
    ap.add_argument("--calibration-copy", action="store_true",
                    help="also launch one plain 256 MiB device copy (k_calibration_copy): the known-size "
                         "launch a rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE reading is scaled by")
    ap.add_argument("--profile-forward", type=int, nargs=2, metavar=("BATCH", "ROWS"), default=None,
                    help="run only the verify forward of the base model at BATCH sequences x ROWS rows "
                         "(200 back-to-back forwards after one verify call) and print its time: the command "
                         "the per-shape rocprofv3 summaries under profiles/ are made with")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on exactly one GPU (no sharding, no collectives); use --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import paper_2205_10350_amd as ad
    from ad_inputs import CONFIGS, SPECIAL, draw_sources, edit_guide, init_weights, model_dims, positional_draft

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    cfg1, cfg2 = CONFIGS[1], CONFIGS[2]
    dims = model_dims(cfg1["model"])
    V = dims["vocab"]
    w = init_weights(dims, cfg1["seed"])
    K_MAX = 72
    conf = ad.make_config(dims, max_batch=32, max_src=64, max_len=64, k_max=K_MAX, dtype="bf16", special=SPECIAL)
    ctx = ad.Context(conf, w)
    if args.no_graphs:
        ctx.set_option(ad.AD_OPT_GRAPHS, 0)
    if args.calibration_copy:
        a = torch.zeros(256 << 20, dtype=torch.uint8, device="cuda")
        b = torch.empty_like(a)
        ad.calibration_copy(b, a)
        torch.cuda.synchronize()
        del a, b

    if args.profile_forward:
        Bp, Rp = args.profile_forward
        assert 1 <= Bp <= 32 and 1 <= Rp <= K_MAX, "--profile-forward: 1..32 sequences, 1..72 rows each"
        rng = np.random.default_rng(7)
        srcs_p = [rng.integers(5, V, size=25).astype(np.int32) for _ in range(Bp)]
        ctx.encode(ad.AD_VERIFIER, srcs_p, max_out=[64] * Bp)
        ctx.verify([[int(t) for t in rng.integers(5, V, size=Rp)] for _ in range(Bp)])
        f_us, v_us, v_b2b = ctx.time_verify_forward(200, back_to_back=True)
        print(json.dumps({"profile_forward": {"batch": Bp, "rows": Bp * Rp, "forward_us": f_us,
                                              "vocab_kernel_in_forward_us": v_us, "vocab_kernel_back_to_back_us": v_b2b}}))
        ctx.close()
        return

    _progress("batch 1")
    # ---------------- batch 1: the headline workload ------------------------------------------
    n_sent = cfg1["n_sent"]
    srcs, max_out = draw_sources(cfg1, V)
    if args.sentences > 0:
        n_sent = min(n_sent, args.sentences)
        srcs, max_out = srcs[:n_sent], max_out[:n_sent]
    greedy_out, guides = [], []
    t0 = time.perf_counter()
    for s, mo in zip(srcs, max_out):
        o, _ = ctx.decode_greedy([s], max_out=[mo])
        greedy_out.append(o[0])
    torch.cuda.synchronize()
    t_greedy = time.perf_counter() - t0
    for i, g in enumerate(greedy_out):
        guides.append(edit_guide(g, cfg1["rate"], cfg1["seed"] + i, V))

    def step(i):
        j = i % n_sent
        return ctx.decode_iad([srcs[j]], [guides[j]], max_out=[max_out[j]])

    for i in range(args.warmup):
        step(i)
    # Every call shape of the timed sentences is replayed from a captured graph in the timed region
    # whatever --warmup says: a graph is built on a shape's third appearance, so each timed sentence
    # is decoded three times beforehand (untimed).
    if not args.no_graphs:
        for rep in range(3):
            for i in range(min(args.steps, n_sent)):
                step(i)
    torch.cuda.synchronize()
    toks = its = rows = 0
    t0 = time.perf_counter()
    for i in range(args.steps):
        o, st = step(i)
        toks += len(o[0]); its += st["iterations"]; rows += st["rows_verified"]
        assert o[0] == greedy_out[i % n_sent], "draft-and-verify output differs from greedy"
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    value = toks / dt
    greedy_tps = sum(len(g) for g in greedy_out) / t_greedy

    # verify forward at the first-iteration shape of a typical sentence (whole guide + sentinel)
    j = int(np.argsort([len(s) for s in srcs])[n_sent // 2])
    ctx.encode(ad.AD_VERIFIER, [srcs[j]], max_out=[max_out[j]])
    draft = (list(guides[j]) + [ad.AD_NEVER])[:int(max_out[j])]
    def as_teams(call):   # whether the verify call's layers went out as one launch, and with them those of the timed forwards
        before = ctx.get_option(ad.AD_OPT_TEAM_LAUNCHES)
        call()
        return ctx.get_option(ad.AD_OPT_TEAM_LAUNCHES) > before
    teams = as_teams(lambda: ctx.verify([draft]))
    M1 = len(draft)
    params = decoder_stream_params(dims)
    kv_bytes = dims["dec_layers"] * 2 * 2 * dims["d_model"] * (M1 + len(srcs[j]))
    fwd_bytes = 2 * params + kv_bytes
    fwd_us, voc_us, voc_b2b_us = ctx.time_verify_forward(50, back_to_back=True)
    # the output-projection kernel reading its matrix from 12 rotating copies (393 MB, more than the
    # 256 MB last-level cache holds): every launch streams from HBM.  In the decode loop the base
    # model's 77 MB of weights stay in that cache from one forward to the next, which is what the
    # back-to-back figure measures.
    voc_cold_us = ctx.time_output_projection(12, 48)
    # output projection + arg max: the [V, d] bf16 matrix once, the M x d bf16 rows once, the
    # per-row partial maxima written once
    voc_bytes = 2 * V * dims["d_model"] + 2 * M1 * dims["d_model"] + 8 * M1 * ((V // 16 + 7) // 8)
    # embedding, seven per decoder layer at this row count (or one for all of them), output projection, arg-max finish
    n_launches = 4 if teams else 3 + dims["dec_layers"] * 7
    how = {True: "the layers as one launch", False: "a launch per stage"}
    # The path's roofline: one verify forward (embedding, six decoder layers, output projection with
    # the fused arg max and its finish) at the first-iteration shape of a typical sentence.
    # achieved = algorithmic bytes (every decoder weight the forward streams, once, plus the key /
    # value rows read) over the forward's duration: HIP events on the library's stream around 50
    # forwards launched back to back, / 50.
    roofline = {"bound": "hbm", "kernel": f"verify forward, base model, batch 1 ({how[teams]})",
                "rows": M1, "us": fwd_us, "algorithmic_bytes": fwd_bytes,
                "achieved": fwd_bytes / (fwd_us * 1e-6) / 1e9, "peak": HBM_PEAK / 1e9, "unit": "GB/s",
                "frac": fwd_bytes / (fwd_us * 1e-6) / HBM_PEAK, "traffic": None if teams else VERIFY_FORWARD_TRAFFIC_BYTES,
                "traffic_source": "no counter run of the layers as one launch" if teams else
                                  "rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of `bench.py --profile-forward 1 25 "
                                  "--calibration-copy`, summed over the forward's launches (profiles/)"}
    # the largest single kernel of that forward (42 % of its algorithmic bytes), context only.
    # `frac` = the matrix streamed from HBM on every launch; the figure with the matrix resident in
    # the last-level cache between launches (as it is in the decode loop) under its own name
    vocab_kernel = {"kernel": "k_gemm_bf16_astat<1, 1, 1, true> (output projection + arg max)", "rows": M1,
                    "algorithmic_bytes": voc_bytes, "us": voc_cold_us,
                    "achieved": voc_bytes / (voc_cold_us * 1e-6) / 1e9, "frac": voc_bytes / (voc_cold_us * 1e-6) / HBM_PEAK,
                    "llc_resident_us": voc_b2b_us, "llc_resident_achieved": voc_bytes / (voc_b2b_us * 1e-6) / 1e9,
                    "llc_resident_frac_of_hbm_peak": voc_bytes / (voc_b2b_us * 1e-6) / HBM_PEAK,
                    "bracketed_in_forward_us": voc_us,
                    "traffic_from_profile": VOCAB_KERNEL_TRAFFIC_BYTES}
    verify_bs1 = {"rows": M1, "us": fwd_us, "algorithmic_MB": fwd_bytes / 1e6,
                  "hbm_frac": fwd_bytes / (fwd_us * 1e-6) / HBM_PEAK, "launches": n_launches}

    _progress("batch 32")
    # ---------------- batch 32 ---------------------------------------------------------------------
    bs32 = None
    roofline_bs32 = None
    if not args.no_bs32:
        srcs2, max_out2 = draw_sources(cfg2, V)
        B = cfg2["batch"]
        batches = [(srcs2[i:i + B], max_out2[i:i + B]) for i in range(0, len(srcs2), B)]
        g2, gd2 = [], []
        t0 = time.perf_counter()
        for ss, mo in batches:
            o, _ = ctx.decode_greedy(ss, max_out=mo)
            g2.append(o)
        torch.cuda.synchronize()
        t_g2 = time.perf_counter() - t0
        for bi, o in enumerate(g2):
            gd2.append([edit_guide(g, cfg2["rate"], cfg2["seed"] + bi * B + b, V) for b, g in enumerate(o)])
        ctx.decode_iad(batches[0][0], gd2[0], max_out=batches[0][1])   # warm
        torch.cuda.synchronize()
        toks2 = its2 = rows2 = 0
        t0 = time.perf_counter()
        for (ss, mo), gd, ref in zip(batches, gd2, g2):
            o, st = ctx.decode_iad(ss, gd, max_out=mo)
            assert o == ref, "batched draft-and-verify output differs from greedy"
            toks2 += sum(len(x) for x in o); its2 += st["iterations"]; rows2 += st["rows_verified"]
        torch.cuda.synchronize()
        dt2 = time.perf_counter() - t0
        ss, mo = batches[0]
        ctx.encode(ad.AD_VERIFIER, ss, max_out=mo)
        drafts = [(list(g) + [ad.AD_NEVER])[:int(m)] for g, m in zip(gd2[0], mo)]
        teams32 = as_teams(lambda: ctx.verify(drafts))
        M32 = sum(len(d) for d in drafts)
        fwd32_us, voc32_us = ctx.time_verify_forward(20)
        flops = 2.0 * M32 * params
        bs32 = {"tokens_per_s": toks2 / dt2, "greedy_tokens_per_s": sum(len(x) for o in g2 for x in o) / t_g2,
                "iterations": its2, "rows_verified": rows2,
                "verify_rows": M32, "verify_us": fwd32_us, "verify_gflop": flops / 1e9,
                "mfma_frac": flops / (fwd32_us * 1e-6) / MFMA_BF16_PEAK,
                # all iterations of the decode (rows shrink as the guides are consumed): flops of every row
                # verified over the whole decode's wall time, encoder and host included
                "decode_mean_rows": rows2 / max(1, its2),
                "decode_mfma_frac": 2.0 * rows2 * params / dt2 / MFMA_BF16_PEAK,
                "vocab_kernel_us": voc32_us,
                "vocab_kernel_mfma_frac": 2.0 * M32 * V * dims["d_model"] / (voc32_us * 1e-6) / MFMA_BF16_PEAK}
        roofline_bs32 = {"bound": "mfma", "kernel": f"verify forward, base model, batch 32 ({how[teams32]})",
                         "rows": M32, "us": fwd32_us, "algorithmic_flops": flops,
                         "achieved": flops / (fwd32_us * 1e-6) / 1e12, "peak": MFMA_BF16_PEAK / 1e12, "unit": "TFLOP/s",
                         "frac": flops / (fwd32_us * 1e-6) / MFMA_BF16_PEAK, "traffic": None}
    _progress("sweeps")
    # ---------------- verify forward against block size and batch size (roofline against rows) -------
    sweeps = None
    if not args.no_next:
        rng = np.random.default_rng(77)
        src_len, blk = 25, 36
        def point(Bs, rows_each):
            ss = [rng.integers(5, V, size=src_len).astype(np.int32) for _ in range(Bs)]
            ctx.encode(ad.AD_VERIFIER, ss, max_out=[64] * Bs)
            ctx.verify([[int(t) for t in rng.integers(5, V, size=rows_each)] for _ in range(Bs)])
            # two measurements of 30 forwards, the lower one (a point is taken right after an encode and
            # a verify call of a new shape; the first measurement after them reads up to 10 % high)
            f_us, _, v_us = min(ctx.time_verify_forward(30, back_to_back=True) for _ in range(2))
            Ms = Bs * rows_each
            kvb = dims["dec_layers"] * 2 * 2 * dims["d_model"] * (Ms + Bs * src_len)
            return {"batch": Bs, "rows": Ms, "forward_us": f_us, "vocab_kernel_us": v_us,
                    "forward_hbm_frac": (2 * params + kvb) / (f_us * 1e-6) / HBM_PEAK,
                    "forward_mfma_frac": 2.0 * Ms * params / (f_us * 1e-6) / MFMA_BF16_PEAK,
                    "vocab_hbm_frac": 2 * V * dims["d_model"] / (v_us * 1e-6) / HBM_PEAK,
                    "vocab_mfma_frac": 2.0 * Ms * V * dims["d_model"] / (v_us * 1e-6) / MFMA_BF16_PEAK}
        sweeps = {"block_size_batch1": [point(1, kk) for kk in (1, 2, 4, 8, 10, 15, 20, 25, 30, 40, 64)],
                  "batch_size_block36": [point(bb, blk) for bb in (1, 2, 4, 8, 16, 32)]}
    ctx.close()

    _progress("deep encoder")
    # ---------------- input-guided decoding, deep encoder + shallow decoder (workload 5) --------------
    deep = None
    if not args.no_next:
        cfg5 = CONFIGS[5]
        dims5 = model_dims(cfg5["model"])
        cx = ad.Context(ad.make_config(dims5, max_batch=1, max_src=64, max_len=64, k_max=K_MAX, dtype="bf16",
                                       special=SPECIAL), init_weights(dims5, cfg5["seed"]))
        s5, mo5 = draw_sources(cfg5, V)
        g5 = []
        cx.decode_greedy([s5[0]], max_out=[mo5[0]])
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for s_, m_ in zip(s5, mo5):
            g5.append(cx.decode_greedy([s_], max_out=[m_])[0][0])
        torch.cuda.synchronize()
        t_g5 = time.perf_counter() - t0
        gd5 = [edit_guide(g, cfg5["rate"], cfg5["seed"] + i, V) for i, g in enumerate(g5)]
        for i in range(8):
            cx.decode_iad([s5[i]], [gd5[i]], max_out=[mo5[i]])
        torch.cuda.synchronize()
        tk5 = it5 = 0
        t0 = time.perf_counter()
        for i in range(len(s5)):
            o, st = cx.decode_iad([s5[i]], [gd5[i]], max_out=[mo5[i]])
            assert o[0] == g5[i], "draft-and-verify output differs from greedy"
            tk5 += len(o[0]); it5 += st["iterations"]
        torch.cuda.synchronize()
        t5 = time.perf_counter() - t0
        j5 = int(np.argsort([len(x) for x in s5])[len(s5) // 2])
        cx.encode(ad.AD_VERIFIER, [s5[j5]], max_out=[mo5[j5]])
        d5 = (list(gd5[j5]) + [ad.AD_NEVER])[:int(mo5[j5])]
        cx.verify([d5])
        f5_us, _, v5_us = cx.time_verify_forward(50, back_to_back=True)
        p5 = decoder_stream_params(dims5)
        deep = {"model": "12 encoder + 2 decoder layers, d1024, 16 heads, FFN 4096, vocab 32000", "batch": 1,
                "sentences": len(s5), "tokens_per_s": tk5 / t5, "greedy_tokens_per_s": tk5 / t_g5,
                "speedup_vs_greedy": t_g5 / t5, "mean_tokens_per_forward": tk5 / max(1, it5),
                "verify_rows": len(d5), "verify_forward_us": f5_us, "verify_algorithmic_MB": 2 * p5 / 1e6,
                "verify_forward_hbm_frac": 2 * p5 / (f5_us * 1e-6) / HBM_PEAK, "vocab_kernel_us": v5_us,
                "vocab_kernel_hbm_frac": 2 * V * dims5["d_model"] / (v5_us * 1e-6) / HBM_PEAK}
        cx.close()

    _progress("block drafting")
    # ---------------- draft-and-verify with the block drafter (workloads 3 and 4) ---------------------
    # The drafter forward runs and is timed inside every iteration; its output is replaced by a
    # positional draft with substitutions at the workload's rate (random weights draft nothing useful).
    gad = None
    if not args.no_gad:
        gad = {}
        for wl, n_take, kw in ((3, 64, dict(max_batch=1, max_src=80, max_len=80)),
                               (4, 16, dict(max_batch=8, max_src=512, max_len=128))):
            cfgw = CONFIGS[wl]
            dimsw = model_dims(cfgw["model"])
            ww = init_weights(dimsw, cfgw["seed"])
            wd = init_weights(dimsw, cfgw["seed"] + 7)
            confw = ad.make_config(dimsw, k_max=cfgw["k"], dtype="bf16", special=SPECIAL, **kw)
            cx = ad.Context(confw, ww, wd)
            srcw, mow = draw_sources(cfgw, dimsw["vocab"], n_sent=n_take)
            Bw = cfgw["batch"]
            groups = [(srcw[i:i + Bw], mow[i:i + Bw]) for i in range(0, len(srcw), Bw)]
            refs, drafts = [], []
            cx.decode_greedy(groups[0][0], max_out=groups[0][1])   # warm
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for ss, mo in groups:
                o, _ = cx.decode_greedy(ss, max_out=mo)
                refs.append(o)
            torch.cuda.synchronize()
            t_gr = time.perf_counter() - t0
            for gi, o in enumerate(refs):
                drafts.append([positional_draft(g, cfgw["rate"], cfgw["seed"] + gi * Bw + b, dimsw["vocab"])[0]
                               for b, g in enumerate(o)])
            cx.decode_gad(groups[0][0], cfgw["k"], use_drafter=True, draft_override=drafts[0], max_out=groups[0][1])   # warm
            torch.cuda.synchronize()
            tk = it = 0
            t0 = time.perf_counter()
            for (ss, mo), D, ref in zip(groups, drafts, refs):
                o, st = cx.decode_gad(ss, cfgw["k"], use_drafter=True, draft_override=D, max_out=mo)
                assert o == ref, "draft-and-verify output differs from greedy"
                tk += sum(len(x) for x in o); it += st["iterations"]
            torch.cuda.synchronize()
            t_gad = time.perf_counter() - t0
            gad[f"workload{wl}"] = {"model": cfgw["model"], "batch": Bw, "sentences": len(srcw), "k": cfgw["k"],
                                    "tokens_per_s": tk / t_gad, "greedy_tokens_per_s": tk / t_gr,
                                    "speedup_vs_greedy": t_gr / t_gad, "iterations": it,
                                    "mean_tokens_per_iteration": tk / max(1, it) / Bw}
            # the same decode under the relaxed verification (GAD++, the paper's two presets): not
            # greedy-identical, so only its rate and acceptance are reported (random-init scores
            # put a substituted token far from the top, so few extra tokens stand; the figure shows
            # what the second pass of the output projection costs)
            for name, beta, tau in (("gadpp_3_1.0", 3, 1.0), ("gadpp_5_3.0", 5, 3.0)):
                cx.set_gadpp(beta, tau)
                cx.decode_gad(groups[0][0], cfgw["k"], use_drafter=True, draft_override=drafts[0], max_out=groups[0][1])
                torch.cuda.synchronize()
                tk2 = it2 = 0
                t0 = time.perf_counter()
                for (ss, mo), D in zip(groups, drafts):
                    o, st = cx.decode_gad(ss, cfgw["k"], use_drafter=True, draft_override=D, max_out=mo)
                    tk2 += sum(len(x) for x in o); it2 += st["iterations"]
                torch.cuda.synchronize()
                t2 = time.perf_counter() - t0
                gad[f"workload{wl}"][name] = {"tokens_per_s": tk2 / t2, "iterations": it2,
                                              "mean_tokens_per_iteration": tk2 / max(1, it2) / Bw}
            cx.set_gadpp(1, 0.0)
            cx.close()

    _progress("calibration")
    # ---------------- measured peaks of this machine (context for the nominal ones) -------------------
    a = torch.zeros(256 << 20, dtype=torch.uint8, device="cuda")
    b = torch.empty_like(a)
    ad.calibration_copy(b, a)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(5):
        ad.calibration_copy(b, a)
    e1.record()
    torch.cuda.synchronize()
    copy_gbps = 5 * 2 * a.numel() / (e0.elapsed_time(e1) * 1e-3) / 1e9
    # (measured here, while the GPU is busy: after the seconds of the CPU baseline its clocks are down)
    mfma_tflops = max(ad.calibration_mfma() for _ in range(3))
    del a, b

    _progress("cpu baseline")
    # ---------------- CPU oracle on this machine's host cores (bounded sample) ----------------------
    cpu = None
    if not args.no_cpu_baseline:
        from oracle import ad_oracle as O
        from threadpoolctl import threadpool_info, threadpool_limits
        pools = threadpool_info()
        cores = max([p.get("num_threads", 1) for p in pools] + [1])
        blas = ", ".join(sorted({f"{p.get('internal_api', '?')} {p.get('version', '')}".strip() for p in pools
                                 if p.get("user_api") == "blas"})) or "numpy's BLAS"
        m = O.Model(dims, w, np.float32, max_pos=160)
        n_cpu = min(args.cpu_sentences, n_sent)
        og = [O.greedy(m, srcs[i], int(max_out[i]), SPECIAL["eos"], SPECIAL["bos"]) for i in range(n_cpu)]
        ogd = [edit_guide(g, cfg1["rate"], cfg1["seed"] + i, V) for i, g in enumerate(og)]

        def run_cpu(n):
            t0 = time.perf_counter()
            ct = 0
            for i in range(n):
                o, _ = O.iad(m, srcs[i], ogd[i], int(max_out[i]), SPECIAL["eos"], SPECIAL["bos"], k_max=K_MAX)
                ct += len(o)
            return ct, time.perf_counter() - t0

        ctoks, cdt = run_cpu(n_cpu)
        # the same oracle with the BLAS held to one thread, on a quarter of the sample
        n_one = max(1, n_cpu // 4)
        with threadpool_limits(limits=1):
            c1toks, c1dt = run_cpu(n_one)
        cpu = {"value": ctoks / cdt, "unit": "tokens/s", "cores": int(cores), "kind": "oracle",
               "value_1_thread": c1toks / c1dt,
               "sample": f"first {n_cpu} sentences of the batch-1 workload, numpy float32 oracle on {blas} with "
                         f"{cores} threads, input-guided decoding incl. encoder ({cdt:.1f} s); one-thread figure on the "
                         f"first {n_one} sentences ({c1dt:.1f} s)"}

    line = {
        "metric": "greedy_identical_tokens_per_s", "value": value, "unit": "tokens/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": dt / args.steps * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": "Transformer-base IAD batch 1 (configs[1]): 6+6 layers, d512, 8 heads, FFN 2048, "
                               "vocab 32000, source len ~N(25,8) in [5,64], guide = greedy output + edits 0.1",
                   "batch": 1, "sentences": min(args.steps, n_sent), "k_max": K_MAX},
        "tokens": toks, "verify_forwards": its, "rows_verified": rows,
        "mean_tokens_per_forward": toks / max(1, its), "mean_rows_per_forward": rows / max(1, its),
        # weights streamed by all verify forwards of the timed decode over its wall time (encoder, host included)
        "decode_hbm_frac": its * 2.0 * params / dt / HBM_PEAK,
        "greedy_tokens_per_s": greedy_tps, "speedup_vs_greedy": value / greedy_tps,
        "verify_forward_bs1": verify_bs1, "bs32": bs32, "gad": gad, "sweeps": sweeps, "deep_encoder": deep,
        "measured_copy_GBps": copy_gbps, "measured_mfma_bf16_TFLOPs": mfma_tflops,
        "vocab_kernel": vocab_kernel,
        "roofline": roofline, "roofline_bs32": roofline_bs32, "cpu_baseline": cpu,
    }
    print(json.dumps(line))


if __name__ == "__main__":
    main()
