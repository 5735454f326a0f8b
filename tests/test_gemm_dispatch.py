"""Which bf16 layer products go to the tiled kernels (ad_gemm_tile.hip), on both sides of each rule.  The figures behind a
rule stand at gemm_tile_takes; the results do not depend on the choice (test_gpu_gemm_tile.py)."""
import ctypes

import pytest

from paper_2205_10350_amd import build

QKV, KV, STORE, RELU, RESID = range(5)


@pytest.fixture(scope="module")
def takes():
    f = getattr(ctypes.CDLL(build.LIB_PATH), "_ZN2ad15gemm_tile_takesEiiibi")   # ad::gemm_tile_takes
    f.restype = ctypes.c_bool
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int]
    return lambda M, N, K, ln, mode: f(M, N, K, ln, mode)


@pytest.mark.parametrize("N,last", [(512, 160), (768, 160), (1024, 128), (1536, 80), (2048, 64)])
def test_k_4096_stays_with_the_kernel_whose_waves_share_k_up_to_two_workgroups_per_cu(takes, N, last):
    assert not takes(last, N, 4096, False, RESID)
    assert takes(last + 1, N, 4096, False, RESID)


@pytest.mark.parametrize("N", [512, 768, 1024, 1536, 2048])
def test_k_2048_leaves_the_eight_wave_workgroups_when_they_need_a_second_round(takes, N):
    last = 32 * (256 // (N // 128))   # rows of one round: N / 128 workgroups per 32 rows on 256 CUs
    assert not takes(519, N, 2048, False, RESID)
    assert takes(520, N, 2048, False, RESID) and takes(1024, N, 2048, False, RESID)
    for M in (1025, 1365, max(1024, last), max(1024, last) + 1, 2048, 2049, 4000):
        assert takes(M, N, 2048, False, RESID) == (M <= 1024 or M > last), M
        if M > 1600:
            assert takes(M, N, 1536, False, RESID) == (M > last), M


def test_k_1024_with_few_columns_stays_with_the_few_row_kernel_up_to_its_160_rows(takes):
    for N in (512, 768):
        assert not takes(160, N, 1024, False, RESID) and takes(161, N, 1024, False, RESID)
    assert not takes(128, 1024, 1024, False, RESID) and takes(129, 1024, 1024, False, RESID)


@pytest.mark.parametrize("N,first", [(1408, 1400), (1536, 1400), (2048, 1025), (2080, 600), (2560, 801), (3072, 513), (4096, 257), (6144, 161)])
def test_k_512_behind_a_layernorm(takes, N, first):
    """2048 and 2560 columns: the rows at which the 16-wave workgroups (256 columns x 32 rows) fill the 256 CUs."""
    mode = QKV if N == 1536 else RELU
    assert not takes(first - 1, N, 512, True, mode) and takes(first, N, 512, True, mode) and takes(4000, N, 512, True, mode)
    for few in (512, 1024, 1280):
        assert not any(takes(M, few, 512, True, RELU) for M in (520, 1025, 1345, 2048, 4000))
