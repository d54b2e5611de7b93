"""FP8 projections with one row per wave (contiguous rows, L > 8): rows around the
four of a workgroup and the 32 of a row block, last groups partly or wholly empty,
16-byte and single-value staging, rounds of 4 to 32 indices and several rounds, a
basis narrower than the pass, and the common path's L = 8 beside it; element by
element against the oracle (bound of test_gpu_gemm)."""
import numpy as np
import pytest

from tests.test_gpu_gemm import _check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pg():
    from paper_1411_2860_amd import projgemm
    projgemm.lib()
    return projgemm


@pytest.mark.parametrize("prec", ["fp8", "fp8x2"])
@pytest.mark.parametrize("L,M,K,W,r", [
    (8, 5, 64 * 8 + 4, 33, 8), (12, 1, 12 * 64, 32, 7), (12, 4, 12 * 65 + 4, 31, 1), (16, 3, 16 * 63 + 1, 65, 8),
    (20, 33, 20 * 10 + 4, 5, 5), (24, 2, 24 * 64 - 2, 64, 8), (32, 31, 32 * 64, 7, 3), (64, 36, 64 * 66 + 8, 29, 8),
    (256, 5, 256 * 3 + 255, 9, 2), (48, 1, 3, 2, 8)])
def test_rows(pg, prec, L, M, K, W, r):
    rng = np.random.default_rng(L + M)
    A = rng.standard_normal((M, K)) * np.exp2(rng.integers(-6, 7, (M, 1)))
    B = rng.standard_normal((K, W))
    kind = "haar" if L & (L - 1) == 0 else "dct2"
    _check(pg, A, B, kind, L, r, prec, transB=True)
