"""Backward with its contractions cut into ranges, and the general synthesis:
ranges added in the synthesis for few projections (rows aligned or not) and by a
kernel of their own (FP32, more projections), an odd number of k-blocks in a
range, one to 256 projections around the synthesis' step of 8.  Closed-form
gradients in FP64 (bounds of test_gpu_backward); the number of ranges is
asserted.  Last, the time of shapes that share all but their alignment or their
number of projections."""
import ctypes

import numpy as np
import pytest

from tests import _ref, _tol
from tests.test_gpu_backward import _grad_bounds
from tests.test_gpu_backward_edges import _check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PREC = {"f32": 1, "bf16": 2, "bf16x3": 3, "f16": 4, "f16x3": 5}


def _ranges(prec, M, K, W, L, r):
    """Ranges that the products for dA and dB are planned with."""
    from paper_1411_2860_amd import projgemm as pg
    f = pg.lib()._ZN2pj15gemm_parts_planEilllPiS0_
    f.restype = None
    KB = 8 if prec == "f32" else 16
    rg = r * -(-(-(-K // L)) // KB) * KB
    out = []
    for P, Q, k in ((M, rg, W), (rg, W, M)):
        cfg, n = ctypes.c_int(), ctypes.c_int()
        f(PREC[prec], ctypes.c_long(P), ctypes.c_long(Q), ctypes.c_long(-(-k // KB)), ctypes.byref(cfg), ctypes.byref(n))
        out.append(n.value)
    return tuple(out)


@pytest.mark.parametrize("prec,M,K,W,L,r,ranges", [
    ("f32", 4096, 600, 768, 8, 7, (1, 8)),          # dB: 512 k-blocks
    ("f32", 1024, 520, 4100, 8, 8, (8, 2)),          # dA: 513 k-blocks, odd ranges
    ("f32", 4096, 512, 4096, 64, 24, (8, 8)),        # summed by a kernel
    ("bf16x3", 1024, 515, 4096, 4, 4, (8, 2)),       # rows of 515: stored value by value
    ("bf16x3", 1024, 512, 4096, 64, 24, (1, 2))])    # planned, not used
def test_ranges(prec, M, K, W, L, r, ranges):
    assert _ranges(prec, M, K, W, L, r) == ranges
    _check(prec, "dct2", M, K, W, L, r, saved=True)


@pytest.mark.parametrize("transA,transB", [(True, False), (False, True), (True, True)])
def test_ranges_transposed(transA, transB):
    _check("f32", "dct2", 1024, 520, 4100, 8, 8, transA, transB, saved=True)
    _check("f16x3", "dct2", 1024, 512, 4096, 4, 3, transA, transB, saved=True)


SYNTHESIS = [(65, 32, 17), (130, 64, 24), (131, 64, 25), (300, 256, 256), (90, 33, 8), (37, 9, 9)]


@pytest.mark.parametrize("K,L,r", SYNTHESIS)
def test_general_synthesis(K, L, r):
    _check("f32", "dct2", 33, K, 70, L, r)


@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 7, 11, 15])
def test_general_synthesis_rest(r):
    """What is left of the projections after steps of 8."""
    _check("f32", "dct2", 33, 70, 40, 15, r)


@pytest.mark.parametrize("K,L,r", SYNTHESIS + [(40, 8, 8), (41, 8, 1)])
def test_general_synthesis_f64(K, L, r):
    from paper_1411_2860_amd import projgemm as pg
    M, W = 33, 70
    rng = np.random.default_rng(K + L)
    A, B, dR = rng.standard_normal((M, K)), rng.standard_normal((K, W)), rng.standard_normal((M, W))
    C, D = _ref.oracle_basis("dct2", L)
    Ad, Bd, dRd = (torch.from_numpy(x).cuda() for x in (A, B, dR))
    dA, dB = pg.gemm_backward(Ad, Bd, dRd, r, pg.Basis("dct2", L), prec="f64")
    torch.cuda.synchronize()
    Q = C[:, :r] @ D[:r, :]
    G = -(-K // L)
    pad = lambda X: np.concatenate([X, np.zeros((G * L - K, X.shape[1]))])
    QB = np.concatenate([Q @ pad(B)[g * L:(g + 1) * L] for g in range(G)])[:K]
    QA = np.concatenate([Q.T @ pad(A.T)[g * L:(g + 1) * L] for g in range(G)])[:K].T
    bA, bB = _grad_bounds(A, B, C, D, r, dR, "f64", L)
    _tol.assert_within(dA.cpu().numpy(), dR @ QB.T, bA, f"dA {(K, L, r)}")
    _tol.assert_within(dB.cpu().numpy(), QA.T @ dR, bB, f"dB {(K, L, r)}")


@pytest.mark.parametrize("K", [4, 61, 62, 63, 127])
def test_unaligned_rows(K):
    for L, r in ((4, 4), (12, 3), (64, 16)):
        _check("f32", "dct2", 9, K, 40, L, r)


def _us(prec, M, K, W, L, r):
    from paper_1411_2860_amd import projgemm as pg
    A, B, dR = (torch.randn(s, device="cuda") for s in ((M, K), (K, W), (M, W)))
    basis = pg.Basis("dct2", L)
    _, saved = pg.gemm_save(A, B, r, basis, prec=prec)
    ws = torch.empty(int(pg.lib().pj_gemm_backward_saved_workspace_bytes(M, W, K, L, r, PREC[prec])),
                     dtype=torch.uint8, device="cuda")
    run = lambda: pg.gemm_backward_saved(saved, dR, r, basis, M, W, K, prec=prec, workspace=ws)
    for _ in range(3):
        run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(10):
            run()
    ts = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        ts.append(a.elapsed_time(b) * 100)
    return float(np.median(ts))


def test_time_unaligned():
    """Three columns fewer move no more bytes: 1.5 for the narrower stores."""
    t, base = _us("bf16", 512, 4093, 4096, 64, 16), _us("bf16", 512, 4096, 4096, 64, 16)
    assert t <= 1.5 * base, (t, base)


def test_time_more_projections():
    """Twice the projections at most double the contractions and the projected
    values; the outputs stay: at most 2.2 times."""
    t, base = _us("bf16", 256, 4096, 4096, 64, 32), _us("bf16", 256, 4096, 4096, 64, 16)
    assert t <= 2.2 * base, (t, base)
