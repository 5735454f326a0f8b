"""Forwards whose layers run as one launch (a team of 32 workgroups on one XCD per group of sequences) against the same
forwards launch by launch: logits, arg maxima, decode states and drafted tokens bit for bit, at the edges of the kernel's row
tiles (16, 17, 32 rows a team), key ranges (64, 65, 128 keys), chunks (five chunks on a team that works on four at a time) and of its range
(33 rows, 129 keys: the launches)."""
import threading

import numpy as np
import pytest
import torch

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights, model_dims

pytestmark = pytest.mark.gpu

DIMS = model_dims("base")
W = {}


def _context(drafter=False, batch=12, max_src=136, max_len=96, k_max=40):
    for s in (7, 8):
        if s not in W:
            W[s] = init_weights(DIMS, s)
    cfg = ad.make_config(DIMS, max_batch=batch, max_src=max_src, max_len=max_len, k_max=k_max, dtype="bf16", special=SPECIAL, debug_logits=True)
    return ad.Context(cfg, W[7], W[8] if drafter else None)


def _launched(ctx, call):
    """How many forwards of call() ran their layers as one launch."""
    before = ctx.get_option(ad.AD_OPT_TEAM_LAUNCHES)
    got = call()
    return ctx.get_option(ad.AD_OPT_TEAM_LAUNCHES) - before, got


def _tokens(rng, n):
    return rng.integers(5, DIMS["vocab"], size=n).astype(np.int32)


@pytest.mark.parametrize("src,rows", [
    ([25], [1]), ([7], [16]), ([1], [17]), ([64], [32]), ([65], [24]), ([128], [9]), ([129], [9]), ([30], [33]),
    ([12, 33, 5], [16, 3, 32]), ([9] * 8, [1, 2, 4, 8, 9, 16, 24, 25]),
    ([20, 3, 40, 8, 15, 16, 17, 33, 1, 64, 50, 2], [5, 1, 17, 1, 2, 16, 3, 7, 1, 1, 6, 4]),     # more sequences than teams
    ([10] * 12, [1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1]),
])
def test_layers_as_one_launch_give_the_bits_of_the_launches(src, rows):
    """Two calls a sequence (the second against a longer prefix, with one sequence sitting out), with every row of the first block
    fed; the encoder runs as one launch where its rows allow (at most 32 a sentence), the decoder at most 32 rows a team and 128 keys."""
    rng = np.random.default_rng(sum(src) + 131 * sum(rows))
    srcs = [_tokens(rng, n) for n in src]
    first = [list(_tokens(rng, n)) for n in rows]
    ctx = _context()
    try:
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            assert ctx.get_option(ad.AD_OPT_TEAMS) == on
            assert _launched(ctx, lambda: ctx.encode(ad.AD_VERIFIER, srcs))[0] == (on and max(src) <= 32)
            n, v = _launched(ctx, lambda: ctx.verify(first, want_verified=True))
            assert n == (on and max(src) <= 128 and max(rows) <= 32)
            out = [v, ctx.debug_logits().view(np.uint32).copy()]
            second = [[] if b == 1 else list(first[b][:1 + b % 3]) for b in range(len(src))]
            n, v = _launched(ctx, lambda: ctx.verify(second))
            assert n == (on and max(src) <= 128)
            out += [v, ctx.debug_logits().view(np.uint32).copy(), ctx.output()]
            got[on] = out
        for x, y in zip(got[0], got[1]):
            if isinstance(x, np.ndarray):
                assert np.array_equal(x, y)
            else:
                for u, v in zip(x, y):
                    assert np.array_equal(u, v)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("name", ["dec.2.ln1.b", "dec.1.self.bk", "dec.4.self.bq", "dec.0.cross.bo", "dec.3.ffn.b1", "dec.3.ffn.b2", "enc.1.self.bv", "enc.2.ffn.b2"])
def test_values_that_are_not_finite_pass_between_the_members(name):
    """A place nobody has written yet is all ones, one of the NaNs: a value of these bits in a bias, as rows, keys, values or hidden units take
    it up, comes through as a NaN (no team gives up), and what stays finite has the bits of the launches."""
    if 7 not in W:
        W[7] = init_weights(DIMS, 7)
    w = dict(W[7])
    w[name] = w[name].copy()
    w[name].view(np.uint32)[77] = 0xffffffff
    rng = np.random.default_rng(len(name))
    srcs = [_tokens(rng, n) for n in (12, 30)]
    blk = [[int(t) for t in _tokens(rng, n)] for n in (6, 20)]
    ctx = ad.Context(ad.make_config(DIMS, max_batch=2, max_src=32, max_len=32, k_max=20, dtype="bf16", special=SPECIAL, debug_logits=True), w)
    try:
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            ctx.encode(ad.AD_VERIFIER, srcs)
            launched, _ = _launched(ctx, lambda: ctx.verify(blk, want_verified=True))
            assert launched == on
            got[on] = ctx.debug_logits().copy()
        there = np.isfinite(got[0])
        assert there.all() == (name == "dec.3.ffn.b1")   # (the ReLU takes a NaN for less than nothing)
        assert np.array_equal(there, np.isfinite(got[1]))
        assert np.array_equal(got[0][there].view(np.uint32), got[1][there].view(np.uint32))
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("n", [64, 65, 128, 129])
def test_team_forwards_against_long_prefixes(n):
    """A block of 8 rows that ends at key n (own keys): the team kernels for 64 and 128 keys, and the launches beyond."""
    rng = np.random.default_rng(n)
    src = [_tokens(rng, 30)]
    ctx = _context(batch=2, max_len=132, k_max=132)
    try:
        ctx.set_option(ad.AD_OPT_TEAMS, 0)
        g = ctx.decode_greedy(src, max_out=[n - 8])[0][0]
        assert len(g) == n - 8   # (another model or source if it ends earlier)
        tail = list(_tokens(rng, 8))
        got = []
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            ctx.encode(ad.AD_VERIFIER, src)
            assert ctx.verify([g])[0][0] == n - 8
            launched, v = _launched(ctx, lambda: ctx.verify([tail], want_verified=True))
            assert launched == (on and n <= 128)
            got.append((v[2], ctx.debug_logits().view(np.uint32).copy()))
        assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    finally:
        ctx.close()


@pytest.mark.parametrize("lens,k", [([9], 4), ([9, 21, 2], 7), ([5] * 9, 3), ([40], 20)])
def test_drafter_as_one_launch(lens, k):
    """Mask rows and prefix rows of a sequence in one team, the last layer for the mask rows only; both encoders side by side."""
    rng = np.random.default_rng(17 * len(lens) + k)
    srcs = [_tokens(rng, n) for n in lens]
    ctx = _context(drafter=True)
    try:
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            out = []
            for _ in range(2):
                ctx.encode(ad.AD_VERIFIER, srcs)
                ctx.encode(ad.AD_DRAFTER, srcs)
                for step in range(3):
                    launched, d = _launched(ctx, lambda: ctx.draft_nat(k).copy())
                    assert launched == on or step > 0
                    out.append(d)
                    out.append(ctx.debug_logits().view(np.uint32).copy())
                    out += list(ctx.verify([list(row[:k]) for row in d]))
            got[on] = out
        for x, y in zip(got[0], got[1]):
            assert np.array_equal(x, y)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("rows", [[17], [32], [20, 3], [17, 32, 18], [32, 17, 25, 20], [16, 17, 1, 1, 1, 1], [25, 25, 25, 25, 1]])
def test_sequences_cut_into_pieces_on_several_xcds(rows):
    """Two to eight teams, the pieces of a sequence reading each other's keys and values, one XCD a team and two that take turns (up to four teams);
    against prefixes of 0 and 40 tokens (own keys in one and in two key ranges), eagerly and replayed; the last: more pieces than XCDs."""
    rng = np.random.default_rng(sum(rows) + len(rows))
    srcs = [_tokens(rng, 8 + 5 * i) for i in range(len(rows))]
    blk = [list(_tokens(rng, r)) for r in rows]
    ctx = _context()
    try:
        ctx.set_option(ad.AD_OPT_TEAMS, 0)
        pre = ctx.decode_greedy(srcs, max_out=[30] * len(rows))[0]
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            out = []
            for _ in range(4):      # (a graph from the third time where the shape has one)
                ctx.encode(ad.AD_VERIFIER, srcs)
                for step in range(2):
                    launched, v = _launched(ctx, lambda: ctx.verify(blk, want_verified=True))
                    assert launched == on
                    out += [v[2], ctx.debug_logits().view(np.uint32).copy()]
                    if step == 0:
                        ctx.encode(ad.AD_VERIFIER, srcs)
                        n, _ = ctx.verify([p[:30] for p in pre])
                        assert list(n) == [30] * len(rows)
            got[on] = out
        for x, y in zip(got[0], got[1]):
            assert np.array_equal(x, y)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("drafter,lens,teams", [
    (False, [25] * 8, 4), (False, [32] * 8, 4), (False, [7] * 12 + [32, 1], 4),   # 17 to 32 rows a team on eight XCDs
    (True, [32] * 4, 4), (True, [20, 31, 29], 4),                                 # on four, beside the other model's
    (True, [30] * 5, 2)])                                                         # on five: until the shape has its graph
def test_encoders_with_more_than_16_rows_a_team(drafter, lens, teams):
    """Four encodings of one shape, other tokens each, the graph of the launches there from the third on: how many go out as teams,
    and the scores of the launches every time."""
    rng = np.random.default_rng(sum(lens))
    ctx = _context(drafter, batch=14, max_src=40, max_len=16, k_max=4)
    try:
        calls = [[_tokens(rng, n) for n in lens] for _ in range(4)]
        got = {}
        for on in (1, 0):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            n, got[on] = 0, []
            for srcs in calls:
                n += _launched(ctx, lambda: ctx.encode(ad.AD_VERIFIER, srcs))[0]
                ctx.verify([[int(s[0])] for s in srcs])
                got[on].append(ctx.debug_logits().view(np.uint32).copy())
            assert n == (teams if on else 0)
        for x, y in zip(got[1], got[0]):
            assert np.array_equal(x, y)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("prefix,k", [(0, 17), (15, 1), (20, 30), (40, 40), (60, 40)])
def test_drafts_of_more_rows_than_a_team_holds(prefix, k):
    """Mask rows and prefix rows of one sequence over 2, 2, 4, 6 and 7 teams, every piece seeing all of them; teams without a mask row
    end after the last layer's keys and values."""
    rng = np.random.default_rng(prefix + k)
    srcs = [_tokens(rng, 21)]
    ctx = _context(drafter=True)
    try:
        ctx.set_option(ad.AD_OPT_TEAMS, 0)
        g = ctx.decode_greedy(srcs, max_out=[96])[0][0]
        assert len(g) == 96
        got = []
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            ctx.encode(ad.AD_VERIFIER, srcs)
            ctx.encode(ad.AD_DRAFTER, srcs)
            for lo in range(0, prefix, 30):
                n, _ = ctx.verify([g[lo:min(lo + 30, prefix)]])
                assert n[0] == min(30, prefix - lo)
            launched, d = _launched(ctx, lambda: ctx.draft_nat(k).copy())
            assert launched == on
            got.append((d, ctx.debug_logits().view(np.uint32).copy()))
        assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


@pytest.mark.parametrize("rows", [[1] * 8 + [17], [17] + [1] * 8, [1] * 4 + [32] + [1] * 4, [1] * 12 + [32], [1] * 31 + [25], [25] + [1] * 31, [1] * 8 + [16, 16]])
def test_one_long_sequence_among_many_short_ones(rows):
    """More than eight sequences cut into few teams, one of them above a row tile (two to four teams, which would leave XCDs over): the encoder over
    sources of these lengths, then the blocks."""
    rng = np.random.default_rng(sum(rows) + 7 * rows[0])
    srcs = [_tokens(rng, n) for n in rows]
    blk = [list(_tokens(rng, n)) for n in rows]
    other = [_tokens(rng, n) for n in rows]
    ctx = _context(batch=32, max_src=40, max_len=40, k_max=32)
    try:
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            ctx.encode(ad.AD_VERIFIER, other)       # (what a forward that does not run would leave behind)
            ctx.verify([b[::-1] for b in blk])
            assert _launched(ctx, lambda: ctx.encode(ad.AD_VERIFIER, srcs))[0] == on
            launched, v = _launched(ctx, lambda: ctx.verify(blk, want_verified=True))
            assert launched == on
            got[on] = [v[2], ctx.debug_logits().view(np.uint32).copy()]
            ctx.verify([b[:1] for b in blk])        # over the keys the block left
            got[on].append(ctx.debug_logits().view(np.uint32).copy())
        for x, y in zip(got[0], got[1]):
            assert np.array_equal(x, y)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


def test_a_team_that_does_not_come_together_leaves_the_call_to_the_launches():
    """The wait of the team's barrier set to nothing: every kernel gives up and exits, the calls are repeated launch by launch (the
    encoders too) with the results they always have, and the launches keep the next calls."""
    rng = np.random.default_rng(5)
    srcs = [_tokens(rng, n) for n in (9, 30, 4)]
    ctx = _context(drafter=True)
    try:
        ref, _ = ctx.decode_greedy(srcs, max_out=[20] * 3)
        ctx.set_option(ad.AD_OPT_TEAMS, 0)
        got = {}
        for wait in (None, 0):
            if wait is not None:
                ctx.set_option(ad.AD_OPT_TEAMS, 1)
                ctx.set_option(ad.AD_OPT_TEAM_WAIT, wait)
            ctx.encode(ad.AD_VERIFIER, srcs)
            ctx.encode(ad.AD_DRAFTER, srcs)
            d = ctx.draft_nat(5).copy()
            dl = ctx.debug_logits().view(np.uint32).copy()
            if wait is not None:
                assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 1
                ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)      # (ends the launches' turn)
            v = ctx.verify([g[:6] for g in ref], want_verified=True)
            got[wait] = [d, dl, *v, ctx.debug_logits().view(np.uint32).copy()]
            out = ctx.output()
            if wait is not None:
                assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 2
                assert out == first
            first = out
        for x, y in zip(got[None], got[0]):
            assert np.array_equal(x, y)
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)              # the next decode's first call fails, the others are launches
        assert ctx.decode_greedy(srcs, max_out=[20] * 3)[0] == ref
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 3
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 30000)
        assert ctx.decode_greedy(srcs, max_out=[20] * 3)[0] == ref
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 3
    finally:
        ctx.close()


@pytest.mark.parametrize("lens", [[9, 30, 4], [12]])
def test_drafts_of_an_encoder_that_gave_up_without_the_watched_ticket(lens):
    """AD_OPT_SPIN_WAIT 0: ad_draft_nat gets its tokens by a copy, and asks there too whether the drafter's encoder (and the
    verifier's, whose memory the next ad_verify reads) came together."""
    rng = np.random.default_rng(50 + len(lens))
    srcs = [_tokens(rng, n) for n in lens]
    ctx = _context(drafter=True)
    try:
        ctx.set_option(ad.AD_OPT_SPIN_WAIT, 0)
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)
        got = []
        for teams in (1, 0):
            ctx.set_option(ad.AD_OPT_TEAMS, teams)
            ctx.encode(ad.AD_VERIFIER, srcs)
            ctx.encode(ad.AD_DRAFTER, srcs)
            d = ctx.draft_nat(5).copy()
            got.append([d, ctx.debug_logits().view(np.uint32).copy(), *ctx.verify([list(row) for row in d]), ctx.debug_logits().view(np.uint32).copy()])
            assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 1
        for x, y in zip(*got):
            assert np.array_equal(x, y)
    finally:
        ctx.close()


def test_timed_forwards_that_give_up_leave_the_cache_as_it_was():
    """ad_time_verify_forward repeats the last forward over accepted rows; where its teams give up, the keys and values it has
    written are replaced, and the next block scores as it does without the timing."""
    rng = np.random.default_rng(60)
    srcs = [_tokens(rng, n) for n in (11, 30)]
    more = [[int(t) for t in _tokens(rng, 6)] for _ in srcs]
    ctx = _context(batch=2)
    try:
        ctx.set_option(ad.AD_OPT_TEAMS, 0)
        ref, _ = ctx.decode_greedy(srcs, max_out=[20] * 2)
        got = []
        for teams, wait in ((0, None), (1, None), (1, 0)):
            ctx.set_option(ad.AD_OPT_TEAMS, teams)
            ctx.encode(ad.AD_VERIFIER, srcs)
            n, _ = ctx.verify([g[:9] for g in ref])
            assert list(n) == [9, 9]
            if wait is not None:
                ctx.set_option(ad.AD_OPT_TEAM_WAIT, wait)
            if teams:
                assert ctx.time_verify_forward(2)[0] > 0
                assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == (0 if wait is None else 1)
                assert ctx.time_verify_forward(1, back_to_back=True)[0] > 0      # (the launches, from here on)
                assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == (0 if wait is None else 1)
            got.append([*ctx.verify(more), ctx.debug_logits().view(np.uint32).copy()])
        for g in got[1:]:
            for x, y in zip(got[0], g):
                assert np.array_equal(x, y)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 1
    finally:
        ctx.close()


def test_setting_the_wait_lets_replayed_graphs_finish():
    """AD_OPT_TEAM_WAIT drops the graphs; ad_encode has returned with one of them queued, on either stream."""
    rng = np.random.default_rng(70)
    srcs = [_tokens(rng, 128) for _ in range(12)]
    ctx = _context(drafter=True)
    try:
        got = []
        for wait in (None, 20000, 30000):
            for _ in range(4):
                ctx.encode(ad.AD_VERIFIER, srcs)
                ctx.encode(ad.AD_DRAFTER, srcs)
            if wait is not None:
                assert ctx.get_option(ad.AD_OPT_GRAPHS_CAPTURED) >= 2
                ctx.set_option(ad.AD_OPT_TEAM_WAIT, wait)
                assert ctx.stream.query() and ctx.get_option(ad.AD_OPT_GRAPHS_CAPTURED) == 0
            d = ctx.draft_nat(4)
            got.append([d.copy(), *ctx.verify([list(row) for row in d]), ctx.debug_logits().view(np.uint32).copy()])
        for g in got[1:]:
            for x, y in zip(got[0], g):
                assert np.array_equal(x, y)
    finally:
        ctx.close()


def test_an_encoding_that_gave_up_is_forgotten_with_the_next():
    """The sentences of an encoding whose teams gave up are replaced, by one that takes no team, before anything asks for them: the next
    results are not taken for results of the old one."""
    rng = np.random.default_rng(90)
    old, new = [_tokens(rng, 9), _tokens(rng, 4)], [_tokens(rng, 12), _tokens(rng, 5)]
    ctx = _context(drafter=True, batch=2)
    try:
        got = []
        for first in (None, old):
            if first is not None:
                ctx.set_option(ad.AD_OPT_TEAMS, 1)
                ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)
                ctx.encode(ad.AD_VERIFIER, first)
                ctx.encode(ad.AD_DRAFTER, first)
            ctx.set_option(ad.AD_OPT_TEAMS, 0)
            ctx.encode(ad.AD_VERIFIER, new)
            ctx.encode(ad.AD_DRAFTER, new)
            d = ctx.draft_nat(4)
            got.append([d.copy(), *ctx.verify([list(row) for row in d]), ctx.debug_logits().view(np.uint32).copy()])
            assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
        for x, y in zip(*got):
            assert np.array_equal(x, y)
    finally:
        ctx.close()


def test_the_launches_turn_gets_shorter_again():
    """Each failure doubles the calls that go without teams; 64 results in a row whose teams came together halve them again."""
    srcs = [_tokens(np.random.default_rng(100), 9)]
    ctx = _context(batch=1)

    def calls():
        ctx.encode(ad.AD_VERIFIER, srcs)
        ctx.verify([[7]])
        return ctx.get_option(ad.AD_OPT_TEAM_FAILURES)

    def until_the_next_failure():
        before = ctx.get_option(ad.AD_OPT_TEAM_FAILURES)
        return next(i for i in range(1, 300) if calls() > before)
    try:
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)
        assert calls() == 1                                # 32 calls (an encoding and a block each time) without teams, then 64
        assert until_the_next_failure() == 16 + 1
        assert until_the_next_failure() == 32 + 1
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 30000)
        for _ in range(3 * 64):
            assert calls() == 3
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)
        assert calls() == 4
        assert until_the_next_failure() == 16 + 1
    finally:
        ctx.close()


def test_a_repeat_does_not_wait_for_the_null_stream():
    """What a call does after its teams gave up stays on the context's stream: work queued on the null stream goes on."""
    rng = np.random.default_rng(80)
    srcs = [_tokens(rng, 9)]
    ctxs = []
    try:
        # (streams share hardware queues: a context whose stream runs beside the null stream is needed)
        for _ in range(4):
            ctxs.append(_context(batch=1))
            ctx = ctxs[-1]
            got = []
            for teams in (0, 1):
                ctx.set_option(ad.AD_OPT_TEAMS, teams)
                ctx.set_option(ad.AD_OPT_TEAM_WAIT, 0)
                torch.cuda.synchronize()
                torch.cuda._sleep(200_000_000)
                end = torch.cuda.Event()
                end.record()
                ctx.encode(ad.AD_VERIFIER, srcs)
                got.append(ctx.verify([[7, 8, 9]]))
                beside = not end.query()
                if not beside:
                    break
            if teams:
                break
        else:
            pytest.skip("no stream of four runs beside the null stream")
        assert beside and ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 1
        assert all(np.array_equal(x, y) for x, y in zip(*got))
    finally:
        torch.cuda.synchronize()
        for ctx in ctxs:
            ctx.close()


def _verify_beside_the_drafters_encoder(ctx, rng, rows, vocab, draft_src=32, passes=6):
    """Blocks verified while the drafter's encoder, on the library's second stream, holds XCDs 4 to 7: the second XCDs of the teams start late.
    -> logits of all blocks, forwards with teams"""
    got, n = [], 0
    for _ in range(passes):
        ctx.encode(ad.AD_VERIFIER, [rng.integers(5, vocab, size=2).astype(np.int32) for _ in rows])
        for beside in (False, True, False):
            blk = [list(rng.integers(5, vocab, size=k).astype(np.int32)) for k in rows]
            if beside:
                ctx.encode(ad.AD_DRAFTER, [rng.integers(5, vocab, size=draft_src).astype(np.int32) for _ in rows])
            launched, _ = _launched(ctx, lambda: ctx.verify(blk))
            n += launched
            got.append(ctx.debug_logits().view(np.uint32).copy())
    return got, n


@pytest.mark.parametrize("rows", [[9, 16, 12, 13], [1, 1, 1, 1], [16, 1, 5], [25, 9], [25, 25]])
def test_the_second_xcd_of_a_team_may_start_late(rows):
    """The first XCD has done its layer long before the second is there, and the places of the second's rows hold those of an earlier forward
    until then: nothing of them is taken (every pass has other tokens), and no team gives up within the wait of 1 ms."""
    ctx = _context(drafter=True, batch=4, max_src=40, max_len=96, k_max=32)
    try:
        ctx.set_option(ad.AD_OPT_TEAM_WAIT, 100000)
        assert ctx.get_option(ad.AD_OPT_OVERLAP_ENCODERS) == 1
        got = {}
        for on in (0, 1):
            ctx.set_option(ad.AD_OPT_TEAMS, on)
            got[on], n = _verify_beside_the_drafters_encoder(ctx, np.random.default_rng(len(rows) + sum(rows)), rows, DIMS["vocab"])
            assert n == 18 * on
        for x, y in zip(got[0], got[1]):
            assert np.array_equal(x, y)
        assert ctx.get_option(ad.AD_OPT_TEAM_FAILURES) == 0
    finally:
        ctx.close()


def test_teams_of_two_contexts_beside_each_other():
    """Forwards of 1 row and of 25 rows from two threads, a stream each, over the same XCDs: the launches' bits whoever comes first."""
    rows = ([1], [25])
    calls = [[list(_tokens(np.random.default_rng(100 * i + j), r[0])) for j in range(24)] for i, r in enumerate(rows)]
    src = [_tokens(np.random.default_rng(9), 8)]
    ctxs = [_context(batch=1, max_src=16, max_len=64, k_max=32) for _ in rows]
    try:
        got = [{}, {}]

        def run(i, on):
            out = []
            for blk in calls[i]:
                ctxs[i].encode(ad.AD_VERIFIER, src)
                ctxs[i].verify([blk])
                out.append(ctxs[i].debug_logits().view(np.uint32).copy())
            got[i][on] = out
        for on in (0, 1):
            for c in ctxs:
                c.set_option(ad.AD_OPT_TEAMS, on)
            threads = [threading.Thread(target=run, args=(i, on)) for i in range(2)]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
        for i in range(2):
            assert len(got[i][1]) == 24
            for x, y in zip(got[i][0], got[i][1]):
                assert np.array_equal(x, y)
            assert ctxs[i].get_option(ad.AD_OPT_TEAM_LAUNCHES) > 0
    finally:
        for c in ctxs:
            c.close()


def test_two_contexts_in_two_threads():
    """Teams of two contexts that want the same compute units at the same time: the same tokens."""
    rng = np.random.default_rng(6)
    srcs = [[_tokens(rng, n) for n in ns] for ns in ((9, 14), (12,))]
    ctxs = [_context(batch=2), _context(batch=2)]
    try:
        ref = []
        for c, s in zip(ctxs, srcs):
            c.set_option(ad.AD_OPT_TEAMS, 0)
            ref.append(c.decode_greedy(s, max_out=[24] * len(s))[0])
            c.set_option(ad.AD_OPT_TEAMS, 1)
        got = [[], []]

        def run(i):
            for _ in range(4):
                got[i].append(ctxs[i].decode_greedy(srcs[i], max_out=[24] * len(srcs[i]))[0])
        threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for i in range(2):
            assert got[i] == [ref[i]] * 4
            assert ctxs[i].get_option(ad.AD_OPT_TEAM_LAUNCHES) > 0
    finally:
        for c in ctxs:
            c.close()
