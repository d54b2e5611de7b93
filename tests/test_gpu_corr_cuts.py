"""Blocks of at most 8 samples: the row cuts of the one-launch correlation (64,
128 and 512 rows a workgroup) on both sides of their lines, with ragged last
tiles, taps that leave waves without a share, and several staged tap tiles;
both rates and both modes, every output against the oracle (bound of
test_gpu_conv)."""
import numpy as np
import pytest

import oracle
from tests import _ref, _tol
from tests.test_gpu_conv import _check, _dev, conv_bound

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pg():
    from paper_1411_2860_amd import projgemm
    projgemm.lib()
    return projgemm


@pytest.mark.parametrize("L,rows,N", [(L, rows, N) for L in range(1, 9)
                                      for rows, N in [(1, 5), (65, 1), (25472, 33), (25473, 70)]] +
                         [(1, 130561, 19), (2, 130561, 19)])
def test_full_rate(pg, L, rows, N):
    rng = np.random.default_rng(L + rows)
    W = rows * L + N - 1
    s, k = rng.standard_normal(W), rng.standard_normal(N)
    for r in sorted({1, L}):
        if pg.conv1d_method_workspace_bytes(W, N, L, r, "direct") != 256:
            pytest.fail("not the one-launch path")
        _check(pg, s, k, "dct2", L, r, mode="xcorr" if r == 1 else "conv")


@pytest.mark.parametrize("L,rows,N", [(2, 30, 7), (2, 9701, 600), (8, 25480, 100), (3, 131000, 10), (4, 2000, 5000)])
def test_block_rate(pg, L, rows, N):
    rng = np.random.default_rng(L + rows)
    W = rows * L + N - 1
    s, k = rng.standard_normal(W), rng.standard_normal(N)
    C, D = _ref.oracle_basis("dct2", L)
    for r in sorted({1, L}):
        y = pg.conv1d(_dev(s), _dev(k), r, pg.Basis("dct2", L), rate="block")
        torch.cuda.synchronize()
        m = np.arange(W - N + 1)
        ref = oracle.xcorr_proj_block_rate_at(s, k, C, D, r, m)
        mag = oracle.xcorr_proj_block_rate_at(np.abs(s), np.abs(k), np.abs(C), np.abs(D), r, m)
        bound = conv_bound(L, r, N, mag) + 4.0 * 3 * _tol.U["f32"] * mag
        _tol.assert_within(y.double().cpu().numpy(), ref, bound, f"block L={L} r={r} N={N}")


def test_direct_long_taps(pg):
    """Several staged tap tiles with 16 waves (direct path asked for)."""
    rng = np.random.default_rng(3)
    s, k = rng.standard_normal(9000), rng.standard_normal(7001)
    for L, r in ((1, 1), (4, 3), (8, 8)):
        C, D = _ref.oracle_basis("dct2", L)
        y = pg.conv1d_method(_dev(s), _dev(k), r, pg.Basis("dct2", L), method="direct")
        torch.cuda.synchronize()
        ref = oracle.xcorr_proj(s, k, C, D, r)
        mag = oracle.xcorr_proj(np.abs(s), np.abs(k), np.abs(C), np.abs(D), r)
        _tol.assert_within(y.double().cpu().numpy(), ref, conv_bound(L, r, k.size, mag), f"long taps L={L}")
