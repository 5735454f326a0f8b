"""The few-row bf16 GEMMs whose waves share K (widths 1024, 2048 and 4096): bit equality with the tiled kernels at every
remainder of a 16-row tile (four rows are requested at a time) and on both sides of each rule of their dispatch.

The sums are the same chain in every kernel (k ascending, 32 at a time, one accumulator), so the bound is equality."""
import numpy as np
import pytest

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights

pytestmark = pytest.mark.gpu

DIMS = {
    "d1024": dict(enc_layers=1, dec_layers=2, d_model=1024, n_heads=16, d_ffn=4096, vocab=2000),
    # FFN2 with K = 2048, FFN1 with half the columns
    "d1024 narrow": dict(enc_layers=1, dec_layers=2, d_model=1024, n_heads=16, d_ffn=2048, vocab=2000),
}
# rows of a call, one sequence after the other filled with up to 72
ROWS = [1, 3, 4, 5, 8, 9, 12, 13, 15, 16, 17, 20, 21, 31, 32, 33, 48, 63, 64, 65, 96, 97, 128, 129, 160, 161]


@pytest.mark.parametrize("name", DIMS)
def test_rows_do_not_depend_on_how_many_share_the_launch(name):
    dims = DIMS[name]
    rng = np.random.default_rng(11)
    cfg = ad.make_config(dims, max_batch=8, max_src=64, max_len=80, k_max=72, dtype="bf16", special=SPECIAL, debug_logits=True)
    srcs = [rng.integers(5, dims["vocab"], size=40).astype(np.int32) for _ in range(8)]
    blocks = [[int(t) for t in rng.integers(5, dims["vocab"], size=72)] for _ in srcs]
    with ad.Context(cfg, init_weights(dims, 12)) as ctx:
        def logits(rows):
            ctx.encode(ad.AD_VERIFIER, srcs)
            ctx.verify([b[:min(72, max(0, rows - 72 * i))] for i, b in enumerate(blocks)])
            return ctx.debug_logits().view(np.uint32)
        many = logits(8 * 72)
        for rows in ROWS:
            assert np.array_equal(logits(rows), many[:rows]), rows
