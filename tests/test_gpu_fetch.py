"""ad_debug_logits brings the scores to the host through a pinned ring of 1 MB slots: one slot, a slot's edge, a partly filled
last slot and more pieces than the ring has slots give the bits that one direct copy (into pinned memory) gives."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights

pytestmark = pytest.mark.gpu
V = 16384   # 64 KB a row: 16 rows are one slot


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 64, 65, 80])
def test_scores_arrive_whole(rows):
    dims = dict(enc_layers=1, dec_layers=1, d_model=64, n_heads=4, d_ffn=128, vocab=V)
    w = init_weights(dims, 3)
    cfg = ad.make_config(dims, max_batch=2, max_src=8, max_len=96, k_max=88, dtype="fp32", special=SPECIAL, debug_logits=True)
    rng = np.random.default_rng(rows)
    with ad.Context(cfg, w) as ctx:
        ctx.encode(ad.AD_VERIFIER, [rng.integers(5, V, 5).astype(np.int32)], max_out=[90])
        ctx.verify([[int(t) for t in rng.integers(5, V, rows)]])
        pin = torch.full((rows, V), float("nan"), pin_memory=True)
        n = C.c_int(0)
        assert ctx.L.ad_debug_logits(ctx.h, C.cast(pin.data_ptr(), C.POINTER(C.c_float)), rows, C.byref(n)) == 0 and n.value == rows
        for _ in range(2):
            got = ctx.debug_logits()
            assert got.shape == (rows, V) and got.flags.owndata and np.isfinite(got).all()
            assert np.array_equal(got.view(np.uint32), pin.numpy().view(np.uint32))
