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
    # an FFN width whose last column tile is ragged
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
