"""Element types in the Python binding: FP64 batches get FP64 outputs, operands of
another type than the precision's are refused before any device work (the kernels
would read or write past them)."""
import numpy as np
import pytest

import oracle
from tests import _ref, _tol

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec,wrong", [("f64", torch.float32), ("f32", torch.float64), ("bf16", torch.float16)])
def test_refused(prec, wrong):
    from paper_1411_2860_amd import projgemm as pg
    right = torch.float64 if prec == "f64" else torch.float32
    basis = pg.Basis("dct2", 4)
    A, B = torch.zeros((8, 8), dtype=right), torch.zeros((8, 8), dtype=right)
    bad = torch.zeros((8, 8), dtype=wrong)
    for call in (lambda: pg.gemm_batched([A, bad], [B, B], 2, basis, prec=prec),
                 lambda: pg.gemm_batched([A], [bad], 2, basis, prec=prec),
                 lambda: pg.gemm_batched([A], [B], 2, basis, prec=prec, outs=[bad]),
                 lambda: pg.gemm_backward(bad, B, A, 2, basis, prec=prec),
                 lambda: pg.gemm_backward(A, B, bad, 2, basis, prec=prec)):
        with pytest.raises(TypeError):
            call()


@pytest.mark.gpu
@pytest.mark.parametrize("transB", [False, True])
def test_f64_batch(transB):
    from paper_1411_2860_amd import projgemm as pg
    L, r = 16, 5
    C, D = _ref.oracle_basis("dct2", L)
    rng = np.random.default_rng(9)
    As = [rng.standard_normal((m, k)) for m, k in ((1, 3), (40, 200), (257, 130))]
    Bs = [rng.standard_normal((a.shape[1], w)) for a, w in zip(As, (5, 300, 131))]
    outs = pg.gemm_batched([torch.from_numpy(a).cuda() for a in As],
                           [torch.from_numpy(np.ascontiguousarray(b.T if transB else b)).cuda() for b in Bs], r,
                           pg.Basis("dct2", L), prec="f64", transB=transB)
    for a, b, out in zip(As, Bs, outs):
        assert out.dtype == torch.float64
        Gp = -(-(-(-a.shape[1] // L)) // 8) * 8
        _tol.assert_within(out.cpu().numpy(), oracle.gemm_proj(a, b, C, D, r),
                           _tol.gemm_bound("f64", L, r, Gp, _tol.magnitude(a, b, C, D, r)), f"{a.shape}")
