"""The calls a user of this framework times: whole decodes and block verifications through `Context`.

A program keeps one `Context` per model (weights on the GPU, workspace, captured graphs) and sends it sentence after
sentence.  A case says which model, how many sentences, how long, and which of the entry points decodes them; a pass is one
call with everything in it: the encoder(s), the decode loop or the one verified block, and the tokens handed back.

The model sizes, source and output lengths, block sizes and draft error rates are those of `ad_inputs`, whose six workloads
the tests and `bench.py` run; weights are random, N(0, 0.02), as there.
"""
import functools
import math

import numpy as np
import torch

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, edit_guide, model_dims, param_spec, positional_draft
from ad_inputs.gen import FIRST_CONTENT

# What a context is created for: the capacities the tests and bench.py give these models.
CAPACITY = {
    ("tiny", False): dict(max_batch=4, max_src=32, max_len=32, k_max=8),
    ("base", False): dict(max_batch=32, max_src=64, max_len=64, k_max=72),
    ("base", True): dict(max_batch=4, max_src=80, max_len=80, k_max=25),
    ("big", True): dict(max_batch=8, max_src=512, max_len=128, k_max=25),
    ("deep_shallow", False): dict(max_batch=4, max_src=64, max_len=64, k_max=72),
}
MODEL_SEED = {"tiny": 1000, "base": 1001, "big": 1004, "deep_shallow": 1005}


def _case(name, call, model, batch, src_lo, src_hi, **more):
    """One case.  call: "greedy", "iad" (input-guided), "gad" (block drafting) or "block" (encode and verify one block).
    out: output tokens per sentence (0: as many as its source has).  k, rate: block size and draft / guide error rate.
    beta, tau: the relaxed verification (beta 1: off).  logits: the rows' scores are fetched too."""
    c = dict(call=call, model=model, dtype="bf16", batch=batch, src_lo=src_lo, src_hi=src_hi, out=0, k=0, rate=0.1,
             drafter=False, beta=1, tau=0.0, logits=False)
    c.update(more)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # The smallest model in fp32 (workload 0): every launch is tiny, so it is launches and host path that count.
        _case("tiny_gad_fp32", "gad", "tiny", 1, 24, 24, dtype="fp32", out=32, k=8),
        # Plain greedy decoding of one sentence, what drafting is compared with: one decoder row per forward.
        _case("base_greedy_b1", "greedy", "base", 1, 25, 25),
        # Grammar correction of one sentence as it is typed (workload 1, the headline figure).
        _case("base_iad_b1", "iad", "base", 1, 27, 27),
        # The same as a batch job (workload 2): ragged lengths, ragged acceptance.
        _case("base_iad_b32", "iad", "base", 32, 10, 60),
        # Translation with the block drafter, one sentence (workload 3).
        _case("base_gad_b1", "gad", "base", 1, 49, 49, k=25, rate=0.3, drafter=True),
        # The same under the relaxed verification with the paper's first preset (top 3, tau 1).
        _case("base_gadpp_b1", "gad", "base", 1, 37, 37, k=25, rate=0.3, drafter=True, beta=3, tau=1.0),
        # Summarisation (workload 4): the wide model, full sources, both models' encoders, outputs of 128 tokens.
        _case("big_gad_b8", "gad", "big", 8, 512, 512, out=128, k=25, rate=0.3, drafter=True),
        # Time to the first accepted tokens of the same job: the encoder over eight long documents of different lengths.
        _case("big_block_b8", "block", "big", 8, 301, 512, out=128, k=25, drafter=True),
        # Grammar correction with the deep-encoder, shallow-decoder model (workload 5).
        _case("deep_iad_b1", "iad", "deep_shallow", 1, 25, 25),
        # One whole batch scored in one forward (the first iteration of workload 2, a rescoring job): many rows, all arg maxima back.
        _case("base_block_b32", "block", "base", 32, 10, 60),
        # One sentence's scores over the vocabulary: what an inspection of the model's predictions fetches.
        _case("base_logits_b1", "block", "base", 1, 25, 25, logits=True),
        # The same model in fp32, a handful of sentences: the reference-precision run.
        _case("base_iad_fp32_b4", "iad", "base", 4, 10, 60, dtype="fp32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("tiny", "greedy", "iad", "iad", "gad", "long", "deep", "block", "logits", "fp32"))
    lo, hi = sorted((_log_int(rng, 5, 64), _log_int(rng, 5, 64)))
    batch = _log_int(rng, 1, 32)
    if kind == "tiny":
        lo, hi = sorted((rng.randint(5, 32), rng.randint(5, 32)))
        return _case(None, rng.choice(("gad", "iad", "greedy")), "tiny", rng.randint(1, 4), lo, hi, k=rng.randint(2, 8),
                     dtype=rng.choice(("fp32", "bf16")))
    if kind in ("greedy", "iad", "block"):
        return _case(None, kind, "base", batch, lo, hi)
    if kind == "gad":
        lo, hi = sorted((rng.randint(20, 80), rng.randint(20, 80)))
        beta, tau = rng.choice(((1, 0.0), (1, 0.0), (3, 1.0), (5, 3.0)))
        return _case(None, "gad", "base", rng.randint(1, 4), lo, hi, k=rng.randint(10, 25), rate=0.3, drafter=True, beta=beta, tau=tau)
    if kind == "long":
        lo, hi = sorted((_log_int(rng, 40, 512), _log_int(rng, 40, 512)))
        call = rng.choice(("gad", "block", "greedy"))
        return _case(None, call, "big", rng.randint(1, 8), lo, hi, out=rng.randint(16, 64), k=rng.randint(10, 25), rate=0.3, drafter=True)
    if kind == "deep":
        return _case(None, rng.choice(("iad", "greedy")), "deep_shallow", rng.randint(1, 4), lo, hi)
    if kind == "logits":
        return _case(None, "block", "base", 1, lo, hi, logits=True, dtype=rng.choice(("bf16", "fp32")))
    return _case(None, rng.choice(("iad", "block")), "base", _log_int(rng, 1, 8), lo, hi, dtype="fp32")


def _weights(model, seed):
    """{name: fp32 host array}, drawn on the GPU: ad_inputs' distribution (matrices and biases N(0, 0.02), gains 1 + N(0, 0.02)),
    wider for the tiny model, as in its tests: at 0.02 its outputs hardly depend on the source."""
    std = 0.15 if model == "tiny" else 0.02
    gen = torch.Generator("cuda").manual_seed(seed)
    out = {}
    for name, shape, kind in param_spec(model_dims(model)):
        w = torch.randn(shape, generator=gen, device="cuda").mul_(std)
        out[name] = (w + 1.0 if kind == "ln_gain" else w).cpu().numpy()
    return out


@functools.lru_cache(maxsize=None)
def _context(model, dtype, drafter, logits):
    """The context such a program keeps: one per model, precision and purpose."""
    cap = dict(CAPACITY[model, drafter])
    if logits or dtype == "fp32":
        cap["max_batch"] = 1 if logits else min(cap["max_batch"], 8)
    cfg = ad.make_config(model_dims(model), dtype=dtype, special=SPECIAL, debug_logits=logits, **cap)
    seed = MODEL_SEED[model]
    return ad.Context(cfg, _weights(model, seed), _weights(model, seed + 7) if drafter else None)


def prepare(case, seed):
    c = case
    ctx = _context(c["model"], c["dtype"], c["drafter"], c["logits"])
    rng = np.random.default_rng(seed)
    vocab = model_dims(c["model"])["vocab"]
    # lengths spread evenly over the range, in random order
    lens = rng.permutation(np.rint(c["src_lo"] + (c["src_hi"] - c["src_lo"]) * (np.arange(c["batch"]) + 0.5) / c["batch"]).astype(np.int64))
    srcs = [rng.integers(FIRST_CONTENT, vocab, size=n).astype(np.int32) for n in lens]
    max_out = np.full(c["batch"], c["out"], np.int32) if c["out"] else lens.astype(np.int32)
    # The guides and drafts stand for a trained model's: the greedy output with errors at the stated rate.
    proposed = None
    if c["call"] != "greedy":
        ctx.set_gadpp(1, 0.0)
        greedy, _ = ctx.decode_greedy(srcs, max_out=max_out)
        if c["call"] != "iad":
            proposed = [positional_draft(g, c["rate"], seed + b, vocab)[0] for b, g in enumerate(greedy)]
        else:
            proposed = [edit_guide(g, c["rate"], seed + b, vocab) for b, g in enumerate(greedy)]
        if c["call"] == "block":
            rows = [min(int(m), c["k"] or int(m), ctx.cfg.k_max) for m in max_out]
            proposed = [([int(t) for t in p] + [ad.AD_NEVER])[:n] for p, n in zip(proposed, rows)]
    return {"case": dict(c), "ctx": ctx, "srcs": srcs, "max_out": max_out, "proposed": proposed}


def _tokens(outs, width):
    """[sentences, width] token ids, -1 past a sentence's end."""
    t = np.full((len(outs), width), -1, np.int32)
    for row, o in zip(t, outs):
        row[:len(o)] = o
    return t


def run(state):
    c, ctx, srcs, max_out = state["case"], state["ctx"], state["srcs"], state["max_out"]
    if c["call"] == "block":
        ctx.encode(ad.AD_VERIFIER, srcs, max_out=max_out)
        accepted, following, verified = ctx.verify(state["proposed"], want_verified=True)
        got = {"accepted": accepted, "next": following, "verified": verified}
        if c["logits"]:
            got["logits"] = ctx.debug_logits()
        return got
    if c["call"] == "greedy":
        outs, _ = ctx.decode_greedy(srcs, max_out=max_out)
    elif c["call"] == "iad":
        outs, _ = ctx.decode_iad(srcs, state["proposed"], max_out=max_out)
    else:
        ctx.set_gadpp(c["beta"], c["tau"])
        outs, _ = ctx.decode_gad(srcs, c["k"], use_drafter=c["drafter"], draft_override=state["proposed"], max_out=max_out)
    return _tokens(outs, ctx.cfg.max_len)


def work(case):
    """Weights cross from memory once per forward (a forward needs the tokens of the one before), and so do the keys and
    values it reads; products count their multiplications and additions over the rows the method feeds, at the mean source length."""
    c, m = case, model_dims(case["model"])
    d, ffn, vocab, esz = m["d_model"], m["d_ffn"], m["vocab"], 2 if case["dtype"] == "bf16" else 4
    n_src = (c["src_lo"] + c["src_hi"]) / 2
    n_out = c["out"] or n_src
    batch, encoders = c["batch"], 2 if c["drafter"] and c["call"] == "gad" else 1
    enc = m["enc_layers"] * (4 * d * d + 2 * d * ffn) + m["dec_layers"] * 2 * d * d
    dec = m["dec_layers"] * (6 * d * d + 2 * d * ffn) + d * vocab
    if c["call"] == "greedy":
        its, rows = n_out, 1
    elif c["call"] == "iad":
        its, rows = 1 + 1.7 * c["rate"] * n_out, n_out / 2          # an edit costs about two iterations; the guide shrinks
    elif c["call"] == "gad":
        its, rows = n_out * c["rate"] / (1 - (1 - c["rate"]) ** c["k"]), c["k"]
    else:
        its, rows = 1, min(c["k"] or n_out, n_out)
    kv_row = m["dec_layers"] * 2 * d * esz
    flops = encoders * batch * n_src * (2 * enc + 4 * m["enc_layers"] * d * n_src)
    flops += its * batch * rows * (2 * dec + 4 * m["dec_layers"] * d * (n_src + n_out / 2))
    byts = encoders * (esz * enc + batch * n_src * kv_row) + its * (esz * dec + batch * (n_src + n_out / 2) * kv_row)
    if encoders == 2:   # the drafter's forward, prefix and masks, before each verification
        flops += its * batch * (n_out / 2 + c["k"]) * (2 * (dec - d * vocab) + 4 * m["dec_layers"] * d * n_src)
        flops += its * batch * c["k"] * 2 * d * vocab
        byts += its * (esz * dec + batch * n_src * kv_row)
    if c["logits"]:
        byts += batch * rows * vocab * 4
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # fp32: sums of up to 2048 products in another order change a score by about 1e-6 of the scores' rms; the two best of a
    # row are seldom that close.  bf16: a rounding of an activation that falls the other way spreads to 1e-3 rms of scores
    # whose rms is 0.45, and decides the row's arg max in 0.6 % of the rows (both observed against a float64 model).
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4} if case["logits"] else "exact"
    return {"rel": 1e-2, "max": 1e-1, "differ": 1e-2}
