"""FP32 contraction on the BF16 matrix cores: odd and even k-block counts,
tile edges, and the values the three-way split cannot carry (infinities, NaN,
values that round to a BF16 infinity, values below 2^-102), whose tiles are
computed with the FP32 instructions.  With L = 1 the projection is the identity,
so the result is the plain product: compared with FP64 element by element,
finite values within the FP32 bound of tests/_tol.py, infinities and NaN equal."""
import numpy as np
import pytest

from tests import _tol

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CFGS = (17, 16, -1)


def _run(A, B, cfg):
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("identity", 1)
    (M, K), W = A.shape, B.shape[1]
    Ad = torch.from_numpy(A).cuda()
    Bd = torch.from_numpy(np.ascontiguousarray(B.T)).cuda()
    if cfg < 0:
        return pg.gemm(Ad, Bd, 1, basis, transB=True).double().cpu().numpy()
    Ap, Bp = pg.pack_ab(Ad, Bd, 1, basis, transB=True)
    buf = torch.full((M, W + 5), 3.0, device="cuda")
    pg.gemm_packed(Ap, Bp, 1, M, W, K, 1, 1, 1, out=buf[:, :W], tile_cfg=cfg)
    assert torch.all(buf[:, W:] == 3.0)
    return buf[:, :W].double().cpu().numpy()


def _check(A, B, cfg, what):
    got = _run(A, B, cfg)
    with np.errstate(all="ignore"):
        a, b = A.astype(np.float64), B.astype(np.float64)
        ref = np.zeros((A.shape[0], B.shape[1]))
        for k in range(A.shape[1]):                      # NaN and infinities as IEEE sums give them
            ref = ref + np.outer(a[:, k], b[k])
        mag = np.abs(a) @ np.abs(b)
        over = np.isinf(ref.astype(np.float32))          # results are FP32: past its range they are infinite
        ref[over] = np.sign(ref[over]) * np.inf
    fin = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)), what
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), what
    assert np.all(np.isfinite(got[fin])), what
    K8 = -(-A.shape[1] // 8) * 8
    bound = _tol.gemm_bound("f32", 1, 1, K8, mag)
    off = np.abs(got - ref)[fin] - np.asarray(bound)[fin]
    assert np.all(off <= 0), (what, float(off.max()))


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("M,W,K", [(1, 1, 1), (33, 129, 8), (300, 140, 24), (257, 257, 63), (128, 256, 80),
                                   (2050, 1100, 136), (640, 3400, 40)])
def test_sizes(M, W, K, cfg):
    rng = np.random.default_rng(M + W + K)
    A = (rng.standard_normal((M, K)) * np.exp(2 * rng.standard_normal((M, K)))).astype(np.float32)
    B = rng.standard_normal((K, W)).astype(np.float32)
    _check(A, B, cfg, (M, W, K, cfg))


def _plant(what, A, B):
    big = np.float32(3.4028235e38)
    if what == "inf":
        A[3, 5], A[200, 0] = np.inf, -np.inf
    elif what == "inf_both":
        A[7, 1], A[7, 2] = np.inf, -np.inf               # inf - inf in row 7
    elif what == "nan":
        B[6, 130] = np.nan
    elif what == "max_masked":                           # largest values against zeros
        A[40, :3], B[:3, :] = -big, 0.0
    elif what == "max":
        A[40, :], A[40, 3], B[3, 9] = 0.0, big, 0.5
    elif what == "tiny":
        A[50, :] *= np.float32(2.0 ** -115)
        B[:, 77] *= np.float32(2.0 ** 60)
    elif what == "denormal":
        A[60, :] = (A[60, :].astype(np.float64) * 2.0 ** -134).astype(np.float32)
        B[:, :] *= np.float32(2.0 ** 80)
    elif what == "range":                                # a row and a column of opposite scales
        s = np.float32(2.0) ** np.linspace(-90, 90, A.shape[1]).round().astype(np.float32)
        A[70, :] *= s
        B[:, 33] /= s


@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("what", ["inf", "inf_both", "nan", "max_masked", "max", "tiny", "denormal", "range"])
def test_special_values(what, cfg):
    rng = np.random.default_rng(11)
    A = rng.standard_normal((1500, 56)).astype(np.float32)
    B = rng.standard_normal((56, 1500)).astype(np.float32)
    _plant(what, A, B)
    _check(A, B, cfg, (what, cfg))
