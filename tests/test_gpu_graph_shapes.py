"""The counts that decide when a call shape gets a graph do not grow with every shape there ever was: after 8192 others a shape that has
come twice is counted anew."""
import numpy as np
import pytest

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights, model_dims

pytestmark = pytest.mark.gpu


def test_shapes_that_do_not_come_back_are_forgotten():
    dims, k_max = model_dims("tiny"), 128
    cfg = ad.make_config(dims, max_batch=2, max_src=8, max_len=160, k_max=k_max, dtype="fp32", special=SPECIAL)
    src = [np.array([5, 6, 7], np.int32)] * 2

    def call(ctx, k0, k1):
        ctx.encode(ad.AD_VERIFIER, src)
        ctx.verify([[5] * k0, [6] * k1])
        return ctx.get_option(ad.AD_OPT_GRAPHS_CAPTURED)
    with ad.Context(cfg, init_weights(dims, 1)) as ctx:
        for _ in range(3):
            held = call(ctx, 3, 2)
        assert held == 2                       # the encoder's shape and this one: three appearances each
        others = [(a, b) for a in range(1, k_max + 1) for b in range(1, a + 1) if a + b > 6]
        assert len(others) >= 8192
        for _ in range(2):
            assert call(ctx, 2, 2) == held     # two of three
        for a, b in others:
            assert call(ctx, a, b) == held
        assert call(ctx, 2, 2) == held and call(ctx, 2, 2) == held
        assert call(ctx, 2, 2) == held + 1
