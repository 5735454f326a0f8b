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


@pytest.mark.parametrize("N,last", [(512, 128), (1024, 64), (2048, 32)])
def test_k_4096_leaves_the_kernel_whose_waves_share_k_while_that_is_one_workgroup_per_cu(takes, N, last):
    assert not takes(last, N, 4096, False, RESID)
    assert takes(last + 1, N, 4096, False, RESID)
