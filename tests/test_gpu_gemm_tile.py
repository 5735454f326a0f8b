"""The tiled bf16 GEMMs (many rows): bit equality with the few-row kernels across every tile shape the row count selects.

A sentence is encoded alone (few rows: the kernels that keep a row's whole K in LDS) and inside batches whose row sums fall
on both sides of each rule of the dispatch, with remainders of every tile height; a verify call after each must give the same
logits bit for bit (the encoder's rows and the memory keys and values of the sentence are all it depends on).  The sums are
the same chain in every kernel (k ascending, 32 at a time, one accumulator), so the bound is equality."""
import numpy as np
import pytest

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights

pytestmark = pytest.mark.gpu

DIMS = {
    "d512": dict(enc_layers=2, dec_layers=4, d_model=512, n_heads=8, d_ffn=2048, vocab=2000),
    "d1024": dict(enc_layers=2, dec_layers=2, d_model=1024, n_heads=16, d_ffn=4096, vocab=2000),
    # an inner dimension other than the widths above: 24 stages of K
    "d1024 narrow": dict(enc_layers=1, dec_layers=1, d_model=1024, n_heads=16, d_ffn=1536, vocab=2000),
}
# rows of the whole batch
SUMS = [65, 81, 129, 161, 257, 401, 513, 521, 626, 1025, 1121, 1345, 1537, 2049, 2500, 3253, 4096]


@pytest.mark.parametrize("name", DIMS)
def test_rows_do_not_depend_on_the_tile_shape(name):
    dims = DIMS[name]
    rng = np.random.default_rng(5)
    cfg = ad.make_config(dims, max_batch=64, max_src=240, max_len=16, k_max=8, dtype="bf16", special=SPECIAL, debug_logits=True)
    first = rng.integers(5, dims["vocab"], size=29).astype(np.int32)
    block = [int(t) for t in rng.integers(5, dims["vocab"], size=8)]
    with ad.Context(cfg, init_weights(dims, 6)) as ctx:
        ctx.encode(ad.AD_VERIFIER, [first])
        ctx.verify([block])
        alone = ctx.debug_logits().view(np.uint32)
        for rows in SUMS:
            rest = rows - len(first)
            n = -(-rest // 72)                      # other sentences of about 72 tokens, their lengths ragged
            lens = [rest // n + (1 if i < rest % n else 0) for i in range(n)]
            others = [rng.integers(5, dims["vocab"], size=k).astype(np.int32) for k in lens]
            at = int(rng.integers(0, n + 1))
            ctx.encode(ad.AD_VERIFIER, others[:at] + [first] + others[at:])
            ctx.verify([[]] * at + [block] + [[]] * (n - at))
            assert np.array_equal(ctx.debug_logits().view(np.uint32), alone), rows


# FFN widths whose last column tile is ragged in every shape that can have one (24.5 and 32.5 tiles of 64 columns, 12.25 and 16.25 of
# 128; widths are multiples of 32), and inner dimensions and widths that only the tiled kernels' general rules cover; the rows of
# the batch select each tile shape in turn (32 x 32, 32 x 64, 64 x 64, 64 x 128 four and two stages ahead, the three rolling ones)
EDGES = {
    "d1024, ffn 1568": (dict(enc_layers=1, dec_layers=1, d_model=1024, n_heads=16, d_ffn=1568, vocab=2000),
                        [97, 129, 321, 641, 1217, 2177, 4417, 6402]),
    "d512, ffn 2080": (dict(enc_layers=1, dec_layers=1, d_model=512, n_heads=8, d_ffn=2080, vocab=2000),
                       [520, 577, 995, 1665, 3393, 4865]),
    "d512, ffn 3072": (dict(enc_layers=1, dec_layers=1, d_model=512, n_heads=8, d_ffn=3072, vocab=2000), [129, 513, 673, 1101, 2401]),
    "d1024, ffn 8192": (dict(enc_layers=1, dec_layers=1, d_model=1024, n_heads=16, d_ffn=8192, vocab=2000), [17, 129, 300, 801, 1101]),
    "d1536": (dict(enc_layers=1, dec_layers=1, d_model=1536, n_heads=24, d_ffn=1536, vocab=2000), [17, 97, 129, 700, 1601, 2049]),
    "d2048": (dict(enc_layers=1, dec_layers=1, d_model=2048, n_heads=32, d_ffn=4096, vocab=2000), [33, 129, 520, 1025]),
}


@pytest.mark.parametrize("name", EDGES)
def test_the_last_rows_and_columns_of_every_tile_shape(name):
    """A sentence that ends the batch, in the last, ragged row tile of every launch, and one that begins it, against the same
    sentence alone."""
    dims, sums = EDGES[name]
    rng = np.random.default_rng(7)
    cfg = ad.make_config(dims, max_batch=96, max_src=80, max_len=16, k_max=8, dtype="bf16", special=SPECIAL, debug_logits=True)
    first = rng.integers(5, dims["vocab"], size=13).astype(np.int32)
    block = [int(t) for t in rng.integers(5, dims["vocab"], size=8)]
    with ad.Context(cfg, init_weights(dims, 8)) as ctx:
        ctx.encode(ad.AD_VERIFIER, [first])
        ctx.verify([block])
        alone = ctx.debug_logits().view(np.uint32)
        for rows in sums:
            rest = rows - len(first)
            n = -(-rest // 72)
            others = [rng.integers(5, dims["vocab"], size=rest // n + (1 if i < rest % n else 0)).astype(np.int32) for i in range(n)]
            for at in (0, n):
                ctx.encode(ad.AD_VERIFIER, others[:at] + [first] + others[at:])
                ctx.verify([[]] * at + [block] + [[]] * (n - at))
                assert np.array_equal(ctx.debug_logits().view(np.uint32), alone), (rows, at)
