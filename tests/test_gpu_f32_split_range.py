"""Where the three-way split of FP32 operands ends: values from 2^-110 up stay on
the BF16 matrix cores (their last part is a subnormal BF16 value), smaller ones
send their tile to the FP32 instructions, early, so that such data costs little
more than the FP32 instructions alone."""
import numpy as np
import pytest

from tests import _tol

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _product(A, B, cfg):
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("identity", 1)
    (M, K), W = A.shape, B.shape[0]
    Ap, Bp = pg.pack_ab(A, B, 1, basis, transB=True)
    return pg.gemm_packed(Ap, Bp, 1, M, W, K, 1, 1, 1, tile_cfg=cfg)


@pytest.mark.parametrize("K", [24, 57, 130, 520])
@pytest.mark.parametrize("low,split", [(-110, True), (-106, True), (-111, False), (-126, False), (-149, False)])
def test_range(low, split, K):
    """Row 5 of the left side lies in [2^low, 2^(low + 1)), every mantissa bit in
    use (subnormals: as many as there are)."""
    rng = np.random.default_rng(K - low)
    A = rng.standard_normal((1800, K)).astype(np.float32)
    B = rng.standard_normal((1300, K)).astype(np.float32)
    A[5] = ((1.0 + rng.random(K)) * 2.0 ** low).astype(np.float32) * rng.choice([-1.0, 1.0], K).astype(np.float32)
    assert np.all(np.abs(A[5]) >= np.float32(2.0 ** low))
    B *= np.float32(2.0 ** 70)
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    bound = _tol.gemm_bound("f32", 1, 1, -(-K // 8) * 8, np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64)).T)
    fp32 = _product(Ad, Bd, 5)
    for cfg in (17, 16):
        got = _product(Ad, Bd, cfg)
        _tol.assert_within(got.double().cpu().numpy(), ref, bound, f"{low} {K} {cfg}")
        # the tiles of row 5 carry the FP32 instructions' bits exactly where they ran
        same = torch.equal(got[:128], fp32[:128])
        assert same == (not split), (low, K, cfg)
        assert not torch.equal(got[256:], fp32[256:])


def _time(fn):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(10):
        fn()
    b.record()
    b.synchronize()
    return a.elapsed_time(b) / 10


def test_cost():
    """A tiny value in every tile, 1024 x 8192 outputs over 1024 indices: the call
    is one pass of the FP32 instructions after the first stages, so within 1.35
    of their copy ring (configuration 18; splitting and both passes: 1.65)."""
    from paper_1411_2860_amd import projgemm as pg
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    M, W, K = 1024, 8192, 1024
    A = torch.randn((M, K), generator=g, device="cuda")
    B = torch.randn((W, K), generator=g, device="cuda")
    A[::64] *= 2.0 ** -120
    basis = pg.Basis("identity", 1)
    Ap, Bp = pg.pack_ab(A, B, 1, basis, transB=True)
    out = torch.empty((M, W), device="cuda")
    run = {c: (lambda c=c: pg.gemm_packed(Ap, Bp, 1, M, W, K, 1, 1, 1, out=out, tile_cfg=c)) for c in (18, -1)}
    for f in run.values():
        _time(f)
    ts = {c: [] for c in run}
    for _ in range(9):
        for c, f in run.items():
            ts[c].append(_time(f))
    ring, auto = (float(np.median(ts[c])) for c in (18, -1))
    assert auto <= 1.35 * ring, (auto, ring)
