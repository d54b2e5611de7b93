"""Frequency-domain correlation at the edges of its kernels: every transform
size, phase groups with a remainder (L not a multiple of 4), L and r on both
sides of the fused projection's limit of 32, a tap count that leaves the last
sample pair half empty, one output row, and outputs that are not 16-byte
aligned.  Every output against the oracle within the transform's bound
(derived in test_gpu_conv.fft_bound)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle                                        # noqa: E402
from tests import _ref, _tol                         # noqa: E402
from tests.test_gpu_conv import _dev, fft_bound      # noqa: E402


@pytest.fixture(scope="module")
def pg():
    from paper_1411_2860_amd import projgemm
    projgemm.lib()
    return projgemm


@pytest.mark.parametrize("W,N,L,r,off", [
    (2000, 129, 1, 1, 0),        # F = 512, one phase
    (9000, 510, 2, 2, 1),        # F = 1024, two phases, odd tap count, output off by one float
    (9001, 1500, 3, 2, 0),       # F = 2048, phase group of 3
    (30000, 6 * 700, 6, 5, 0),   # F = 4096, groups of 4 and 2
    (40000, 33 * 20, 33, 33, 0), # signal rows by the tiled pass (L and r above 32)
    (40000, 32 * 20, 32, 32, 2), # fused projection at its limit, output off by two floats
    (12345, 8 * 300 + 1, 8, 3, 0),
    (4100, 4096, 4, 4, 0),       # two output rows
])
@pytest.mark.parametrize("mode", ["xcorr", "conv"])
def test_fft_edges(pg, W, N, L, r, off, mode):
    rng = np.random.default_rng(W + N + L)
    s, k = rng.standard_normal(W), rng.standard_normal(N)
    basis = pg.Basis("dct2", L)
    C, D = _ref.oracle_basis("dct2", L)
    buf = torch.full((W - N + 1 + off + 4,), 7.0, dtype=torch.float32, device="cuda")
    y = pg.conv1d_fft(_dev(s), _dev(k), r, basis, mode=mode, out=buf[off:off + W - N + 1])
    torch.cuda.synchronize()
    kk = k[::-1] if mode == "conv" else k
    ref = oracle.xcorr_proj(s, kk, C, D, r)
    mag = oracle.xcorr_proj(np.abs(s), np.abs(kk), np.abs(C), np.abs(D), r)
    _tol.assert_within(y.double().cpu().numpy(), ref, fft_bound(s, kk, C, D, L, r, mag), f"fft L={L} r={r} N={N}")
    assert torch.all(buf[:off] == 7.0) and torch.all(buf[off + W - N + 1:] == 7.0)
