"""The attention kernel that stages keys and values once per 128 query rows (bf16, head width 64, more than 64 keys or
rows): capacities with one accumulation chain (below 256 keys), with four accumulators, and those whose last keys are a fifth
super-block (beyond 512), with key counts on both sides of every super-block and row counts of several workgroups.

Bounds: bits against the other attention kernels and launch shapes (the order of a sum depends on the key's index alone), the
mode's stated tolerance (2e-2) against the float64 oracle over the bf16-rounded weights."""
import numpy as np
import pytest

import paper_2205_10350_amd as ad
from ad_inputs import SPECIAL, init_weights
from oracle import ad_oracle as O

pytestmark = pytest.mark.gpu


def _dims(d):
    return dict(enc_layers=1, dec_layers=2, d_model=d, n_heads=d // 64, d_ffn=512, vocab=2000)


@pytest.mark.parametrize("cap", [250, 300, 526])
def test_self_attention_and_encoder_rows_against_the_oracle_and_across_blocks(cap):
    dims = _dims(512)
    w = init_weights(dims, 51)
    km = cap - 16
    cfg = ad.make_config(dims, max_batch=4, max_src=cap, max_len=16, k_max=km, dtype="bf16", special=SPECIAL, debug_logits=True)
    rng = np.random.default_rng(52)
    lens = [cap, 129, 200, 128]
    srcs = [rng.integers(5, 2000, size=n).astype(np.int32) for n in lens]
    blocks = [[int(t) for t in rng.integers(5, 2000, size=km)] for _ in lens]
    m = O.Model(dims, {k: (O.bf16_round(v) if v.ndim == 2 else v) for k, v in w.items()}, np.float64, max_pos=cap + 1)
    with ad.Context(cfg, w) as ctx:
        def logits(sel, rows):
            ctx.encode(ad.AD_VERIFIER, [srcs[b] for b in sel])
            ctx.verify([blocks[b][:n] for b, n in zip(sel, rows)])
            return ctx.debug_logits()
        whole = {}
        for b in range(4):   # every row of a block as long as the self-attention's capacity allows
            whole[b] = logits([b], [km])
            want = m.decode_full(m.encode(srcs[b]), [SPECIAL["bos"]] + blocks[b][:km - 1])
            assert np.abs(whole[b] - want).max() < 2e-2, b
        # the same rows in blocks that end elsewhere in a 16-row tile, a super-block or a workgroup, alone and in a batch
        for rows in (1, 16, 65, 127, 128, 129, km - 1):
            got = logits([0], [rows])
            assert np.array_equal(got.view(np.uint32), whole[0][:rows].view(np.uint32)), rows
        rows = [127, km, 1, 130]
        got, r0 = logits([3, 0, 2, 1], rows), 0
        for b, n in zip([3, 0, 2, 1], rows):
            assert np.array_equal(got[r0:r0 + n].view(np.uint32), whole[b][:n].view(np.uint32)), b
            r0 += n


@pytest.mark.parametrize("d", [512, 1024])
@pytest.mark.parametrize("cap", [250, 300, 526])
def test_cross_attention_rows_do_not_depend_on_the_kernel(d, cap):
    """One launch with the query projection (7 rows: the kernel whose waves split the keys where the capacity is 256 or more;
    40 rows at width 512: several tiles per workgroup) against projection and k_attention_rows as two launches."""
    dims = _dims(d)
    rng = np.random.default_rng(61)
    lens = [cap, 127, 128, 129, cap - 1, 65, min(cap, 513), min(cap, 385)]
    srcs = [rng.integers(5, 2000, size=n).astype(np.int32) for n in lens]
    blocks = [[int(t) for t in rng.integers(5, 2000, size=40)] for _ in lens]
    cfg = ad.make_config(dims, max_batch=8, max_src=cap, max_len=16, k_max=40, dtype="bf16", special=SPECIAL, debug_logits=True)
    with ad.Context(cfg, init_weights(dims, 62)) as ctx:
        def logits(fuse, rows):
            ctx.set_option(ad.AD_OPT_FUSE_CROSSQ, fuse)
            ctx.encode(ad.AD_VERIFIER, srcs)
            ctx.verify([b[:rows] for b in blocks])
            return ctx.debug_logits().view(np.uint32).reshape(8, rows, -1)
        want = logits(0, 40)
        assert np.array_equal(logits(1, 40), want)
        for rows in (1, 7, 16, 17):
            assert np.array_equal(logits(1, rows), want[:, :rows]), rows
            assert np.array_equal(logits(0, rows), want[:, :rows]), rows
