"""The grouped contraction's stream of steps across items: more large tiles than
workgroups, items of one, odd and even numbers of k-blocks next to each other
(a step rounded up past the end of an item, a k-block below 0 in its last
step), large and small tiles in one launch.  Every output against the closed
form A Q_r B in FP64 within the rounding bound of tests/_tol.py."""
import numpy as np
import pytest

import oracle
from tests import _ref
from tests import _tol
from tests.test_gpu_batched import _bound

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(2000, 2300, 70), (40, 70, 33), (1800, 2100, 16), (2049, 1025, 330), (300, 500, 700), (257, 129, 257)]


@pytest.fixture(scope="module")
def batch():
    rng = np.random.default_rng(17)
    return [(rng.standard_normal((m, k)), rng.standard_normal((k, w))) for m, w, k in SHAPES]


@pytest.mark.parametrize("prec", ["f32", "bf16", "bf16x3", "f16"])
@pytest.mark.parametrize("cfg,r", [(-1, 3), (16, 1), (17, 3), (18, 2)])
def test_stream_across_items(batch, prec, cfg, r):
    from paper_1411_2860_amd import projgemm as pg
    L = 4
    basis = pg.Basis("dct2", L)
    C, D = _ref.oracle_basis("dct2", L)
    Ad = [torch.from_numpy(a).float().cuda() for a, _ in batch]
    Bd = [torch.from_numpy(b).float().cuda() for _, b in batch]
    outs = [torch.full((a.shape[0], b.shape[1] + 3), 5.0, device="cuda") for a, b in batch]
    pg.gemm_batched(Ad, Bd, r, basis, prec=prec, tile_cfg=cfg, outs=[o[:, :-3] for o in outs])
    torch.cuda.synchronize()
    for i, ((A, B), R) in enumerate(zip(batch, outs)):
        ref = oracle.gemm_proj_closed(A, B, C, D, r)
        _tol.assert_within(R[:, :-3].double().cpu().numpy(), ref, _bound(prec, A, B, C, D, r, L),
                           f"{SHAPES[i]} {prec} cfg={cfg} r={r}")
        assert torch.all(R[:, -3:] == 5.0)
