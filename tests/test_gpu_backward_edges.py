"""The backward's kernels at their edges: dR packed in both orders at once or in
one, contractions in several ranges whose partials the synthesis adds, the
synthesis kernels for few projections (L = 4 .. 256, groups that end past K,
more groups than a workgroup holds, r around 4, 8 and 16, odd leading
dimensions) against the general one (r = 17, L not a multiple of 4).  Closed-form
gradients in FP64, bounds of test_gpu_backward."""
import numpy as np
import pytest

import oracle
from tests import _ref, _tol
from tests.test_gpu_backward import _dev, _grad_bounds

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(prec, kind, M, K, W, L, r, transA=False, transB=False, need=(True, True), saved=False):
    from paper_1411_2860_amd import projgemm as pg
    rng = np.random.default_rng(M + K + W + L + r)
    A, B, dR = rng.standard_normal((M, K)), rng.standard_normal((K, W)), rng.standard_normal((M, W))
    basis = pg.Basis(kind, L)
    C, D = _ref.oracle_basis(kind, L)
    Ad, Bd, dRd = _dev(A.T if transA else A), _dev(B.T if transB else B), _dev(dR)
    if saved:
        _, sv = pg.gemm_save(Ad, Bd, r, basis, prec=prec, transA=transA, transB=transB)
        dA, dB = pg.gemm_backward_saved(sv, dRd, r, basis, M, W, K, prec=prec, transA=transA, transB=transB,
                                        need_dA=need[0], need_dB=need[1])
    else:
        dA, dB = pg.gemm_backward(Ad, Bd, dRd, r, basis, prec=prec, transA=transA, transB=transB, need_dA=need[0],
                                  need_dB=need[1])
    torch.cuda.synchronize()
    Q = C[:, :r] @ D[:r, :]
    G = -(-K // L)
    pad = lambda X: np.concatenate([X, np.zeros((G * L - K, X.shape[1]))])
    QB = np.concatenate([Q @ pad(B)[g * L:(g + 1) * L] for g in range(G)])[:K]
    QA = np.concatenate([Q.T @ pad(A.T)[g * L:(g + 1) * L] for g in range(G)])[:K].T
    bA, bB = _grad_bounds(A, B, C, D, r, dR, prec, L)
    what = (prec, kind, M, K, W, L, r, transA, transB, need, saved)
    if need[0]:
        g = dA.double().cpu().numpy()
        _tol.assert_within(g.T if transA else g, dR @ QB.T, bA, f"dA {what}")
    else:
        assert dA is None
    if need[1]:
        g = dB.double().cpu().numpy()
        _tol.assert_within(g.T if transB else g, QA.T @ dR, bB, f"dB {what}")
    else:
        assert dB is None


@pytest.mark.parametrize("need", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
def test_one_or_both_gradients(need, prec):
    for M, W in ((1, 1), (63, 65), (64, 128), (130, 33)):
        _check(prec, "dct2", M, 48, W, 16, 3, need=need)
        _check(prec, "dct2", M, 48, W, 16, 3, need=need, saved=True)


@pytest.mark.parametrize("transA,transB", [(False, False), (True, True)])
@pytest.mark.parametrize("K,L,r", [(52, 4, 4), (53, 4, 1), (600, 4, 3), (130, 12, 9), (127, 12, 12), (257, 256, 16),
                                   (200, 64, 5), (70, 16, 8), (99, 20, 17), (77, 7, 5), (33, 32, 16)])
def test_synthesis(K, L, r, transA, transB):
    _check("f32", "dct2", 37, K, 301, L, r, transA, transB)


@pytest.mark.parametrize("prec,M,K,W,L,r", [("bf16x3", 1024, 512, 4096, 4, 4), ("f32", 4096, 600, 640, 8, 7),
                                            ("f16x3", 2100, 512, 4000, 4, 2)])
def test_ranges(prec, M, K, W, L, r):
    _check(prec, "dct2", M, K, W, L, r)
