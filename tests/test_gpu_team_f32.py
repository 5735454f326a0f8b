"""fp32 forwards whose layers run as one launch (teams of 32 workgroups, an XCD each) against the same forwards launch by launch, bit for bit: both
widths the kernel has, one to eight teams, pieces of a sequence that read each other's keys, one XCD a team and two by turns, key ranges
of one and of two classes, and what stays with the launches (more than 32 rows of a sequence, more than eight teams, 129 keys)."""
import numpy as np
import pytest

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights, model_dims

pytestmark = pytest.mark.gpu

MODELS = {"d128": dict(model_dims("tiny"), dec_layers=3), "d512": dict(enc_layers=2, dec_layers=3, d_model=512, n_heads=8, d_ffn=2048, vocab=2000)}
W = {}


def _context(model, batch, weights=None, **more):
    if model not in W:
        W[model] = init_weights(MODELS[model], 21)
    cfg = ad.make_config(MODELS[model], max_batch=batch, max_src=136, max_len=96, k_max=40, dtype="fp32", special=SPECIAL, debug_logits=True, **more)
    return ad.Context(cfg, weights or W[model])


def _launched(ctx, call):
    before = ctx.get_option(ad.AD_OPT_TEAM_LAUNCHES)
    got = call()
    return ctx.get_option(ad.AD_OPT_TEAM_LAUNCHES) - before, got


# sources, rows, whether the layers are one launch: width 128, width 512 (where few full teams are left to the launches)
@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("src,rows,teams", [
    ([25], [1], (1, 1)), ([7], [16], (1, 0)), ([1], [17], (1, 0)), ([64], [32], (1, 0)), ([65], [24], (1, 0)), ([65], [8], (1, 1)), ([128], [8], (1, 1)),
    ([129], [8], (0, 0)), ([30], [33], (0, 0)), ([12, 33, 5], [16, 3, 32], (1, 1)), ([70, 5], [32, 31], (1, 1)), ([9] * 4, [16, 2, 13, 1], (1, 1)),
    ([9] * 8, [1, 2, 4, 8, 9, 16, 5, 3], (1, 0)), ([20, 3, 40, 8, 15, 16, 17, 33, 1], [5, 1, 7, 1, 2, 16, 3, 7, 1], (1, 0)), ([6] * 9, [16] * 9, (0, 0)),
    ([10] * 12, [1] * 12, (1, 0)),
])
def test_layers_as_one_launch_give_the_bits_of_the_launches(model, src, rows, teams):
    """A block, a second one against the prefix the first left (one sequence sitting out), and one against 40 tokens more."""
    rng = np.random.default_rng(sum(src) + 131 * sum(rows))
    v = MODELS[model]["vocab"]
    srcs = [rng.integers(5, v, size=n).astype(np.int32) for n in src]
    first = [list(rng.integers(5, v, size=n).astype(np.int32)) for n in rows]
    ctx = _context(model, len(src))
    try:
        ctx.set_option(ad.AD_OPT_TEAMS, 0)
        g = ctx.decode_greedy(srcs, max_out=[40] * len(src))[0]
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            out = []
            for prefix in (0, 40):
                for _ in range(3):      # (a graph from the third time where the shape has one)
                    ctx.encode(ad.AD_VERIFIER, srcs)
                    if prefix:
                        ctx.verify([p[:40] for p in g])
                    live = [b for b in range(len(src)) if not prefix or len(g[b]) == 40]
                    blk = [f if b in live else [] for b, f in enumerate(first)]
                    if not live:
                        continue
                    n, a = _launched(ctx, lambda: ctx.verify(blk, want_verified=True))
                    if not prefix:
                        assert n == (on and teams[model == "d512"])
                    out += [a[0], a[2], ctx.debug_logits().view(np.uint32).copy()]
                    if not prefix:
                        a = ctx.verify([[] if b == 1 else list(first[b][:1 + b % 3]) for b in range(len(src))])
                        out += [a[0], ctx.debug_logits().view(np.uint32).copy(), ctx.output()]
            got[on] = out
        assert len(got[0]) == len(got[1])
        for x, y in zip(got[0], got[1]):
            if isinstance(x, np.ndarray):
                assert np.array_equal(x, y)
            else:
                assert all(np.array_equal(p, q) for p, q in zip(x, y))
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("lens,teams", [([1], (1, 1)), ([8], (1, 1)), ([16], (1, 0)), ([17], (1, 0)), ([32], (1, 0)), ([32, 30], (1, 1)), ([30, 20, 32], (1, 1)), ([8] * 8, (1, 1)),
                                        ([16] * 8, (1, 1)), ([32] * 5, (0, 0))])
def test_encoders_as_one_launch(model, lens, teams):
    rng = np.random.default_rng(sum(lens))
    srcs = [rng.integers(5, MODELS[model]["vocab"], size=n).astype(np.int32) for n in lens]
    ctx = _context(model, len(lens))
    try:
        got = []
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            assert _launched(ctx, lambda: ctx.encode(ad.AD_VERIFIER, srcs))[0] == (on and teams[model == "d512"])
            ctx.set_option(ad.AD_OPT_TEAMS, 0)
            ctx.verify([[7, 8, 9]] * len(lens))
            got.append(ctx.debug_logits().view(np.uint32).copy())
        assert np.array_equal(got[0], got[1])
    finally:
        ctx.close()


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("name", ["dec.1.ln1.b", "dec.0.self.bv", "dec.2.cross.bq", "dec.1.ffn.b1", "enc.1.self.bk"])
def test_values_that_are_not_finite_pass_between_the_members(model, name):
    """All ones, the bits of a place nobody has written yet, as a bias: comes through as a NaN, and what stays finite has the launches' bits."""
    if model not in W:
        W[model] = init_weights(MODELS[model], 21)
    w = dict(W[model])
    w[name] = w[name].copy()
    w[name].view(np.uint32)[77] = 0xffffffff
    rng = np.random.default_rng(len(name))
    srcs = [rng.integers(5, MODELS[model]["vocab"], size=n).astype(np.int32) for n in (12, 30)]
    blk = [[int(t) for t in rng.integers(5, MODELS[model]["vocab"], size=n)] for n in (20, 26)]
    ctx = _context(model, 2, w)
    try:
        got = []
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            ctx.encode(ad.AD_VERIFIER, srcs)
            assert _launched(ctx, lambda: ctx.verify(blk, want_verified=True))[0] == on
            got.append(ctx.debug_logits().copy())
        there = np.isfinite(got[0])
        assert np.array_equal(there, np.isfinite(got[1]))
        assert np.array_equal(got[0][there].view(np.uint32), got[1][there].view(np.uint32))
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


# (an encoder long enough to be in the way)
LATE = {"d128": dict(model_dims("tiny"), enc_layers=6, dec_layers=5), "d512": dict(enc_layers=4, dec_layers=5, d_model=512, n_heads=8, d_ffn=2048, vocab=2000)}


@pytest.mark.parametrize("model", LATE)
@pytest.mark.parametrize("rows", [[9, 16, 12, 13], [1, 1, 1, 1], [8, 1, 5], [25, 9]])
def test_the_second_xcd_of_a_team_may_start_late(model, rows):
    """Blocks verified while the drafter's encoder, on the library's second stream, holds XCDs 4 to 7: the places of the second XCD's rows
    hold those of an earlier forward until it is there, and nothing of them is taken (every pass has other tokens)."""
    dims, key = LATE[model], "late " + model
    if key not in W:
        W[key] = init_weights(dims, 22), init_weights(dims, 23)
    cfg = ad.make_config(dims, max_batch=4, max_src=16, max_len=96, k_max=32, dtype="fp32", special=SPECIAL, debug_logits=True)
    ctx = ad.Context(cfg, *W[key])
    try:
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 100000)
        assert ctx.get_option(ad.AD_OPT_OVERLAP_ENCODERS) == 1
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            rng = np.random.default_rng(len(rows) + sum(rows))
            got[on], n = [], 0
            for _ in range(6):
                ctx.encode(ad.AD_VERIFIER, [rng.integers(5, dims["vocab"], size=2).astype(np.int32) for _ in rows])
                for beside in (False, True, False):
                    blk = [list(rng.integers(5, dims["vocab"], size=k).astype(np.int32)) for k in rows]
                    if beside:
                        assert _launched(ctx, lambda: ctx.encode(ad.AD_DRAFTER, [rng.integers(5, dims["vocab"], size=16 if len(rows) == 4 else 8).astype(np.int32) for _ in rows]))[0] == on
                    n += _launched(ctx, lambda: ctx.verify(blk))[0]
                    got[on].append(ctx.debug_logits().view(np.uint32).copy())
            assert n == on * (18 if model == "d128" or max(rows) <= 16 else 0)   # (width 512: four teams, or teams of at most eight rows)
        for x, y in zip(got[0], got[1]):
            assert np.array_equal(x, y)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("model", MODELS)
def test_a_team_that_does_not_come_together_leaves_the_call_to_the_launches(model):
    rng = np.random.default_rng(5)
    srcs = [rng.integers(5, MODELS[model]["vocab"], size=n).astype(np.int32) for n in (7, 8)]
    ctx = _context(model, 2)
    try:
        ctx.set_option(ad.AD_OPT_TEAMS, 0)
        ref = ctx.decode_greedy(srcs, max_out=[12, 12])[0]
        ctx.set_option(ad.AD_OPT_TEAMS, 1)
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)
        assert ctx.decode_greedy(srcs, max_out=[12, 12])[0] == ref
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) >= 1
    finally:
        ctx.close()
