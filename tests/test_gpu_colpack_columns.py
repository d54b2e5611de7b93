"""Transposed sources of single calls where they go column by column (4 MB and
more): one to four chunks a block, several rounds, lane vectors whole (many
columns) and shared, r = 1, groups that end past K, two sides at once.  The packed
bytes equal the tile packer's on the same values stored with rows contiguous, for
every format of FP32 input; FP64 products match the closed form.  That the
sizes go column by column is asserted with the library's own rule."""
import ctypes

import numpy as np
import pytest

import oracle
from tests import _ref, _tol

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PREC = {"f64": 0, "f32": 1, "bf16": 2, "bf16x3": 3, "f16": 4, "f16x3": 5}


def _columns(prec, P, K, L, r, aligned, split=0):
    from paper_1411_2860_amd import projgemm as pg
    f = pg.lib()._ZN2pj16pack_columns_payEilliiii
    f.restype = ctypes.c_bool
    return f(PREC[prec], ctypes.c_long(P), ctypes.c_long(K), L, r, aligned, split)


# rows, K, L; leading dimension rows + 3: single-value loads in the tile packer.  K is
# a multiple of 4 (16-byte loads of the contiguous copy, the same rounds in both)
SIZES = [(1100, 1200, 4), (1100, 1024, 64), (1024, 1024, 16), (520, 2048, 256), (11000, 96, 48), (13000, 320, 8),
         (1103, 1004, 16), (35000, 60, 32)]


@pytest.mark.parametrize("prec", ["f32", "bf16", "bf16x3", "f16", "f16x3"])
@pytest.mark.parametrize("rows,K,L", SIZES)
def test_same_bytes_as_rows(rows, K, L, prec):
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("dct2", L)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + K)
    X = torch.randn((rows, K), generator=g, device="cuda")
    Xt = torch.zeros((K, rows + 3), device="cuda")[:, :rows]
    Xt.copy_(X.t())
    assert rows * K * 4 >= 4e6
    for r in sorted({1, 2, min(L, 5), min(L, 16), min(L, 19)}):
        assert _columns(prec, rows, K, L, r, 0)
        n = pg.packed_bytes(rows, K, L, r, prec)
        a, b = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
        pg.pack_a(X, r, basis, prec=prec, out=a)
        pg.pack_a(Xt, r, basis, prec=prec, transA=True, out=b)
        assert torch.equal(a, b), (rows, K, L, r, prec)


@pytest.mark.parametrize("M,W,K,L,r,transA", [(40, 1500, 700, 16, 5, False), (700, 1100, 900, 12, 12, True),
                                              (900, 40, 1201, 64, 17, True), (33, 2600, 403, 8, 1, False)])
def test_f64_products(M, W, K, L, r, transA):
    """One side or both (transA) as columns; the first is split between the packers."""
    from paper_1411_2860_amd import projgemm as pg
    rng = np.random.default_rng(M + W)
    A, B = rng.standard_normal((M, K)), rng.standard_normal((K, W))
    C, D = _ref.oracle_basis("dct2", L)
    assert (K * W if not transA else K * (M + W)) * 8 >= 4e6
    R = pg.gemm(torch.from_numpy(A.T.copy() if transA else A).cuda(), torch.from_numpy(B).cuda(), r, pg.Basis("dct2", L),
                prec="f64", transA=transA)
    Gp = -(-(-(-K // L)) // 8) * 8
    _tol.assert_within(R.cpu().numpy(), oracle.gemm_proj(A, B, C, D, r),
                       _tol.gemm_bound("f64", L, r, Gp, _tol.magnitude(A, B, C, D, r)), f"{(M, W, K, L, r)}")


@pytest.mark.parametrize("prec", ["f32", "bf16x3", "f16"])
@pytest.mark.parametrize("P,K,L,r", [(4096, 4096, 64, 8), (4096, 4096, 32, 32), (4104, 4096, 12, 5), (1024, 4096, 256, 16),
                                     (2048, 2048, 64, 16)])
def test_either_packer(P, K, L, r, prec):
    """Aligned sources on both sides of the rule: the bytes do not depend on it."""
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("dct2", L)
    g = torch.Generator(device="cuda")
    g.manual_seed(P + L)
    X = torch.randn((K, P), generator=g, device="cuda")
    Y = torch.zeros((K, P + 1), device="cuda")[:, :P]
    Y.copy_(X)
    n = pg.packed_bytes(P, K, L, r, prec)
    a, b = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    pg.pack_b(X, r, basis, prec=prec, out=a)
    pg.pack_b(Y, r, basis, prec=prec, out=b)          # not aligned: columns
    assert torch.equal(a, b)


def _us(fn):
    for _ in range(3):
        fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(20):
            fn()
    ts = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        ts.append(a.elapsed_time(b) * 50)
    return float(np.median(ts))


@pytest.mark.parametrize("M,W,K,L,r", [(508, 603, 4128, 256, 3), (560, 2240, 2736, 32, 5), (400, 72, 2621, 32, 3)])
def test_pair_time(M, W, K, L, r):
    """Two transposed sources go by one packer: a column more on each (rows no longer
    aligned: columns, one launch) moves the same bytes, 1.3 for the spread."""
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("dct2", L)

    def time(m, w):
        A, B = torch.randn((K, m), device="cuda"), torch.randn((K, w), device="cuda")
        oa, ob = (torch.empty(pg.packed_bytes(x, K, L, r), dtype=torch.uint8, device="cuda") for x in (m, w))
        run = lambda: pg.pack_ab(A, B, r, basis, transA=True, out_a=oa, out_b=ob)
        return _us(run)

    t, base = time(M, W), time(M + 1, W + 1 + W % 2)
    assert t <= 1.3 * base, (t, base)
