"""The fp32 mode's kernels at the edges of their tiles: widths that leave a wave of the K split short or without work,
LayerNorm widths of every load rule, every head width, row counts on both sides of each launch shape's limit.

Bound: an fp32 sum of n products in any order is within n ulp of the float64 one; through two layers of width up to 1024
that stays below 1e-4 for the unit-variance rows and N(0, 0.02) weights used here (the mode's stated tolerance)."""
import numpy as np
import pytest

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights
from oracle import ad_oracle as O

pytestmark = pytest.mark.gpu

MODELS = {
    "d32 heads of 16": dict(enc_layers=1, dec_layers=2, d_model=32, n_heads=2, d_ffn=96, vocab=48),
    "d96 heads of 32": dict(enc_layers=1, dec_layers=1, d_model=96, n_heads=3, d_ffn=160, vocab=1008),
    "d160 no fused norm": dict(enc_layers=1, dec_layers=1, d_model=160, n_heads=5, d_ffn=64, vocab=2000),
    "d256 heads of 128": dict(enc_layers=1, dec_layers=1, d_model=256, n_heads=2, d_ffn=512, vocab=2000),
    "d1024 heads of 64": dict(enc_layers=1, dec_layers=1, d_model=1024, n_heads=16, d_ffn=1056, vocab=2000),
    "d512 wide vocabulary": dict(enc_layers=1, dec_layers=1, d_model=512, n_heads=8, d_ffn=2048, vocab=32000),
}


@pytest.mark.parametrize("name", MODELS)
def test_fp32_rows_against_the_oracle_and_across_launch_shapes(name):
    dims = MODELS[name]
    B, km = 4, 70
    w = init_weights(dims, 11)
    cfg = ad.make_config(dims, max_batch=B, max_src=70, max_len=48, k_max=km, dtype="fp32", special=SPECIAL, debug_logits=True)
    rng = np.random.default_rng(12)
    srcs = [rng.integers(5, dims["vocab"], size=n).astype(np.int32) for n in (1, 17, 33, 70)]
    # blocks of rows: their sums (1, 16, 17, 33, 71, 141, 207) select every launch shape (of the counting pass:
    # test_gpu_vocab_rows.py)
    sizes = [[1], [16], [17], [1, 32], [16, 17, 38], [1, 2, 68, 70], [70, 1, 66, 70]]
    m = O.Model(dims, w, np.float64, max_pos=160)
    seen = {}
    with ad.Context(cfg, w) as ctx:
        for ks in sizes:
            n = len(ks)
            ctx.encode(ad.AD_VERIFIER, srcs[:n])
            fed = [[int(t) for t in np.random.default_rng(100 + b).integers(5, dims["vocab"], size=70)] for b in range(n)]
            _, _, ver = ctx.verify([f[:k] for f, k in zip(fed, ks)], want_verified=True)
            lg = ctx.debug_logits()
            assert lg.shape[0] == sum(ks)
            r0 = 0
            for b, k in enumerate(ks):
                own = lg[r0:r0 + k]
                if b not in seen:
                    seen[b] = (m.decode_full(m.encode(srcs[b]), [SPECIAL["bos"]] + fed[b][:69]), {})
                assert np.abs(own - seen[b][0][:k]).max() < 1e-4, (ks, b)
                assert np.array_equal(ver[b, :k], own.argmax(axis=1)), (ks, b)
                for i in range(k):   # the same bits whichever launch shape served the row
                    bits = seen[b][1].setdefault(i, own[i].view(np.uint32))
                    assert np.array_equal(bits, own[i].view(np.uint32)), (ks, b, i)
                r0 += k


@pytest.mark.parametrize("dh", [16, 32, 64, 128])
def test_fp32_rows_do_not_feel_values_that_are_not_finite_behind_them(dh):
    """A token whose embedding overflows gives keys and values that are not finite; the rows of the block before it must
    keep their bits (a row's keys end at its own: equality), wherever in a 16-row tile and a 16-key unit it stands."""
    dims = dict(enc_layers=1, dec_layers=2, d_model=128, n_heads=128 // dh, d_ffn=128, vocab=512)
    w = init_weights(dims, 21)
    bad = 300
    w["emb"][bad] = 3e38
    cfg = ad.make_config(dims, max_batch=1, max_src=32, max_len=48, k_max=40, dtype="fp32", special=SPECIAL, debug_logits=True)
    rng = np.random.default_rng(22)
    src = rng.integers(5, 300, size=19).astype(np.int32)
    good = [int(t) for t in rng.integers(5, 300, size=40)]
    with ad.Context(cfg, w) as ctx:
        def rows(block):
            ctx.encode(ad.AD_VERIFIER, [src])
            ctx.verify([block])
            return ctx.debug_logits()
        want = rows(good)
        assert np.isfinite(want).all()
        for at in (0, 1, 6, 14, 15, 16, 30, 38):   # the token of row at + 1
            got = rows(good[:at] + [bad] + good[at + 1:])
            assert not np.isfinite(got[at + 1:]).any(), at
            assert np.array_equal(got[:at + 1].view(np.uint32), want[:at + 1].view(np.uint32)), at


@pytest.mark.parametrize("dh", [32, 64])
def test_fp32_attention_over_many_keys(dh):
    """Key ranges of up to 500 (head width 64: 270, about what the configuration check admits), several 16-row tiles, self-attention
    over a long prefix and cross-attention over long sources, against the oracle."""
    dims = dict(enc_layers=1, dec_layers=1, d_model=128, n_heads=128 // dh, d_ffn=128, vocab=512)
    cap = 500 if dh == 32 else 270
    w = init_weights(dims, 31)
    cfg = ad.make_config(dims, max_batch=2, max_src=cap, max_len=20, k_max=cap - 20, dtype="fp32", special=SPECIAL, debug_logits=True)
    rng = np.random.default_rng(32)
    srcs = [rng.integers(5, 512, size=n).astype(np.int32) for n in (cap, 129)]
    blocks = [[int(t) for t in rng.integers(5, 512, size=n)] for n in (cap - 20, 150)]
    m = O.Model(dims, w, np.float64, max_pos=cap + 1)
    with ad.Context(cfg, w) as ctx:
        ctx.encode(ad.AD_VERIFIER, srcs)
        ctx.verify(blocks)
        lg, r0 = ctx.debug_logits(), 0
        for s, b in zip(srcs, blocks):
            want = m.decode_full(m.encode(s), [SPECIAL["bos"]] + b[:-1])
            assert np.abs(lg[r0:r0 + len(b)] - want).max() < 1e-4
            r0 += len(b)
