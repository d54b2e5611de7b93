"""Blocks of at most 8 samples at the lines between 64, 128 and 512 rows a
workgroup (16384 rows, 65536 and, from L = 4, 98304), last tile full and of one row:
every output at the full rate against the oracle (bound of test_gpu_conv)."""
import numpy as np
import pytest

from tests.test_gpu_conv import _check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,r,rows", [(L, r, rows + d) for d in (0, 1) for L, r, rows in
                                      [(1, 1, 16384), (3, 2, 16384), (8, 8, 16384), (1, 1, 65536), (2, 1, 65536),
                                       (4, 1, 98304), (5, 2, 98304)]])
def test_lines(L, r, rows):
    from paper_1411_2860_amd import projgemm as pg
    rng = np.random.default_rng(L + rows)
    N = 23
    W = rows * L + N - 1
    s, k = rng.standard_normal(W), rng.standard_normal(N)
    assert pg.conv1d_method_workspace_bytes(W, N, L, r, "direct") == 256        # the one-launch path
    _check(pg, s, k, "dct2", L, r, mode="xcorr")
