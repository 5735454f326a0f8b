"""Output projection (arg max, and the counting variant of the relaxed verification) at the row counts where its launch
shape changes: a sequence's tokens in a batch of that many rows are its tokens alone, exactly."""
import numpy as np
import pytest

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights

pytestmark = pytest.mark.gpu

# 64 rows end the few-row shape; beyond, 16, 32 and 64 rows per workgroup (the cost model's choice) with several counts of strips
SUMS = [64, 65, 127, 128, 129, 192, 193, 256, 257, 321]
# fp32: 16 rows end the 16 x 32 shape, 48 (1536 tiles) the 32 x 32 one
SUMS_F32 = [1, 16, 17, 32, 33, 48, 49, 100, 144]


def tokens_alone_and_in_batches(dims, dtype, beta, tau, sums):
    rng = np.random.default_rng(41)
    B = 11
    V = dims["vocab"]
    cfg = ad.make_config(dims, max_batch=B, max_src=16, max_len=40, k_max=32, dtype=dtype, special=SPECIAL)
    srcs = [rng.integers(5, V, size=9 + b % 5).astype(np.int32) for b in range(B)]
    with ad.Context(cfg, init_weights(dims, 12)) as ctx:
        ctx.set_gadpp(1, 0.0)
        blocks = []
        for s in srcs:   # the greedy output with an error now and then, so that verification accepts some of it
            g = ctx.decode_greedy([s], max_out=np.array([32], np.int32))[0][0]
            g = [int(t) for t in g] + [int(t) for t in rng.integers(5, V, size=32)]
            blocks.append([t if rng.random() > 0.1 else int(rng.integers(5, V)) for t in g[:32]])
        ctx.set_gadpp(beta, tau)
        for rows in sums:
            n = -(-rows // 32)
            part = [rows // n + (1 if b < rows % n else 0) for b in range(n)]
            mine = [blocks[b][:part[b]] for b in range(n)]
            ctx.encode(ad.AD_VERIFIER, srcs[:n])
            acc, nxt, ver = ctx.verify(mine, want_verified=True)
            for b in range(n):
                ctx.encode(ad.AD_VERIFIER, srcs[b:b + 1])
                a1, n1, v1 = ctx.verify([mine[b]], want_verified=True)
                assert acc[b] == a1[0] and nxt[b] == n1[0], (rows, b)
                assert np.array_equal(ver[b, :part[b]], v1[0, :part[b]]), (rows, b)


@pytest.mark.parametrize("d", [512, 1024])
@pytest.mark.parametrize("beta,tau", [(1, 0.0), (3, 1.0)])
def test_tokens_do_not_depend_on_the_rows_of_the_output_projection(d, beta, tau):
    dims = dict(enc_layers=1, dec_layers=1, d_model=d, n_heads=d // 64, d_ffn=512, vocab=8016)   # 501 strips: ragged in every shape
    tokens_alone_and_in_batches(dims, "bf16", beta, tau, SUMS)


@pytest.mark.parametrize("beta,tau", [(1, 0.0), (3, 1.0), (5, 3.0)])
def test_fp32_tokens_do_not_depend_on_the_rows_of_the_output_projection(beta, tau):
    """The counting launches (a drafted token's score against every column's) in each of their shapes too: a score that differed
    in a bit from the counted column's would count it or drop it."""
    dims = dict(enc_layers=1, dec_layers=1, d_model=256, n_heads=4, d_ffn=256, vocab=8016)
    tokens_alone_and_in_batches(dims, "fp32", beta, tau, SUMS_F32)
