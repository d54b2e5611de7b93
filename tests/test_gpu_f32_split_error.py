"""Rounding of the FP32 contraction on the BF16 matrix cores against that of the
FP32 instructions (the 64 x 64 tile, configuration 5) on the same operands, both
against FP64: dense rows, rows with one value in ten not zero, few groups (so
that a matrix instruction adds only a few terms), positive values.  The root
mean square of the error, in units of 2^-24 of the sum of magnitudes, is no larger
than that of the FP32 instructions (2 % for the sample).  Rows with one value that
is not zero: at most 2.1 units, from one rounding of the sum (1), the products m l'
and l m' (|m| <= 2^-8, |l| <= 2^-17 of the value: 2 x 2^-25 = 1 unit) and the roundings
of the smaller sum (2^-8 of the value each: below 0.1).  The identity basis keeps
the packed values equal to the inputs."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P, Q = 2100, 1060                                     # 17 x 9 tiles of 128 x 128
CFGS = (17, 16, -1)


def _values(what, rows, K, g):
    x = torch.randn((rows, K), generator=g, device="cuda")
    if what == "positive":
        x = x.abs() + 0.01
    if what == "sparse":
        x = x * (torch.rand((rows, K), generator=g, device="cuda") < 0.1)
    if what == "single":
        keep = torch.zeros_like(x)
        keep.scatter_(1, torch.randint(0, K, (rows, 1), generator=g, device="cuda"), 1.0)
        x = x * keep
    return x


def _errors(what, L, K, r, cfgs):
    """(max, rms) per configuration."""
    from paper_1411_2860_amd import projgemm as pg
    g = torch.Generator(device="cuda")
    g.manual_seed(K + r)
    A, B = _values(what, P, K, g), _values("positive" if what == "positive" else "dense", Q, K, g)
    kept = torch.arange(K, device="cuda") % L < r
    a, b = A[:, kept].double(), B[:, kept].double()
    ref, mag = a @ b.t().contiguous(), a.abs() @ b.abs().t().contiguous()
    basis = pg.Basis("identity", L)
    Ap, Bp = pg.pack_ab(A, B, r, basis, transB=True)
    out = []
    for cfg in cfgs:
        R = pg.gemm_packed(Ap, Bp, r, P, Q, K, L, r, r, tile_cfg=cfg)
        e = (R.double() - ref).abs() / (mag + 1e-300) * 2.0 ** 24
        out.append((float(e.max()), float((e * e).mean().sqrt())))
    return out


@pytest.mark.parametrize("what,L,K,r", [
    ("dense", 1, 2, 1), ("dense", 1, 17, 1), ("dense", 1, 40, 1), ("dense", 1, 600, 1), ("sparse", 1, 40, 1),
    ("sparse", 1, 520, 1), ("positive", 1, 300, 1), ("dense", 64, 64, 3), ("dense", 64, 64, 64), ("dense", 64, 128, 2),
    ("positive", 64, 128, 64), ("positive", 64, 64, 16), ("dense", 16, 144, 16)])
def test_no_larger_than_fp32_instructions(what, L, K, r):
    fp32, *split = _errors(what, L, K, r, (5,) + CFGS)
    for cfg, (_, rms) in zip(CFGS, split):
        assert rms <= 1.02 * fp32[1], (what, L, K, r, cfg, rms, fp32[1])


@pytest.mark.parametrize("K", [1, 24, 200])
def test_single_terms(K):
    for cfg, (worst, _) in zip(CFGS, _errors("single", 1, K, 1, CFGS)):
        assert worst <= 2.1, (K, cfg, worst)


@pytest.mark.parametrize("K", [531, 541])
def test_long_ragged(K):
    """1000 x 8200 outputs over 67 and 68 k-blocks, the last partly padding: both split
    tiles and the default, every output, the columns past the last untouched."""
    from paper_1411_2860_amd import projgemm as pg
    from tests import _tol
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    M, W = 1000, 8200
    A = torch.randn((M, K), generator=g, device="cuda")
    B = torch.randn((W, K), generator=g, device="cuda")
    ref = A.double() @ B.double().t().contiguous()
    mag = A.double().abs() @ B.double().abs().t().contiguous()
    Ap, Bp = pg.pack_ab(A, B, 1, pg.Basis("identity", 1), transB=True)
    for cfg in CFGS:
        buf = torch.full((M, W + 3), 7.0, device="cuda")
        pg.gemm_packed(Ap, Bp, 1, M, W, K, 1, 1, 1, out=buf[:, :W], tile_cfg=cfg)
        off = (buf[:, :W].double() - ref).abs() - _tol.gemm_bound("f32", 1, 1, -(-K // 8) * 8, mag)
        assert bool((off <= 0).all()), (cfg, float(off.max()))
        assert bool((buf[:, W:] == 7.0).all())
