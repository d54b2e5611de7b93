"""Packed bytes are a function of the input alone, rows past the last of its row
block included (they are zero), whichever packer writes them: buffers that held
something else before are overwritten in full."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16", "bf16x3", "f16", "f16x3", "fp8", "fp8x2"])
@pytest.mark.parametrize("rows,K,L,r", [(1101, 1008, 16, 5), (35, 200, 8, 3), (4097, 256, 64, 8), (1025, 2048, 8, 1)])
def test_every_byte(rows, K, L, r, prec):
    from paper_1411_2860_amd import projgemm as pg
    basis = pg.Basis("dct2", L)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    X = torch.randn((rows, K), generator=g, device="cuda", dtype=torch.float64 if prec == "f64" else torch.float32)
    for src, trans in ((X, False), (X.t().contiguous(), True)):
        n = pg.packed_bytes(rows, K, L, r, prec)
        bufs = [torch.full((n,), v, dtype=torch.uint8, device="cuda") for v in (0, 0xA5)]
        for b in bufs:
            pg.pack_a(src, r, basis, prec=prec, transA=trans, out=b)
        assert torch.equal(*bufs), (rows, K, L, r, prec, trans)
