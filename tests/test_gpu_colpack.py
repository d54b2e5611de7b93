"""Transposed sources packed column-wise: columns past a tile of 64 or 256,
contraction lengths that end inside a group or a lane vector, blocks whose
matrix-core order has one to four chunks and several rounds, few and many
workgroups (lane vectors whole or shared), leading dimensions larger than the
row.  The packed bytes equal those of the same source stored with its rows
contiguous and aligned alike (the tile packer), bit for bit, for every
matrix-core precision; the product of the FP64 path matches the closed form."""
import numpy as np
import pytest

import oracle
from tests import _ref, _tol

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# L up to 16 or a multiple of 16: the row packer's rounds then add in the same
# order (other L are cut into rounds of their own in each packer, and the two have
# always differed in the last bit there)
SIZES = [(32, 8, 4), (320, 1024, 64), (64, 200, 12), (288, 4096, 8), (1024, 128, 16), (32, 2048, 256), (8192, 96, 48)]


@pytest.mark.parametrize("prec", ["f32", "bf16", "bf16x3", "f16", "f16x3"])
@pytest.mark.parametrize("rows,K,L", SIZES)
def test_same_bytes_as_rows(rows, K, L, prec):
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("dct2", L)
    rng = np.random.default_rng(rows + K)
    X = torch.from_numpy(rng.standard_normal((rows, K)).astype(np.float32)).cuda()
    Xt = torch.zeros((K, rows + 3), device="cuda")[:, :rows]
    Xt.copy_(X.t())
    for r in sorted({2, min(L, 5), min(L, 16), min(L, 19), L}):
        n = pg.packed_bytes(rows, K, L, r, prec)
        a, b = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
        pg.pack_a(X, r, basis, prec=prec, out=a)
        pg.pack_a(Xt, r, basis, prec=prec, transA=True, out=b)
        torch.cuda.synchronize()
        assert torch.equal(a, b), (rows, K, L, r, prec)


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("M,W,K,L,r", [(1, 1, 3, 4, 2), (33, 257, 67, 4, 1), (65, 63, 129, 8, 8), (40, 300, 1000, 12, 5),
                                       (96, 40, 60, 20, 16), (300, 50, 192, 24, 19), (130, 70, 90, 64, 17)])
def test_ragged_products(M, W, K, L, r, prec):
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("dct2", L)
    C, D = _ref.oracle_basis("dct2", L)
    rng = np.random.default_rng(M + W + K)
    A, B = rng.standard_normal((M, K)), rng.standard_normal((K, W))
    dt = torch.float64 if prec == "f64" else torch.float32
    R = pg.gemm(torch.from_numpy(A.T.copy()).to(dt).cuda(), torch.from_numpy(B).to(dt).cuda(), r, basis, prec=prec,
                transA=True)
    torch.cuda.synchronize()
    KB = 16 if prec == "bf16x3" else 8
    Gp = -(-(-(-K // L)) // KB) * KB
    A32, B32 = (A, B) if prec == "f64" else (A.astype(np.float32).astype(np.float64), B.astype(np.float32).astype(np.float64))
    bound = _tol.gemm_bound(prec, L, r, Gp, _tol.magnitude(A32, B32, C, D, r))
    _tol.assert_within(R.double().cpu().numpy(), oracle.gemm_proj(A32, B32, C, D, r), bound, f"{prec} {(M, W, K, L, r)}")
