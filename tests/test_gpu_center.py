"""Centring at the sizes where the number of images held changes: mean (summed
in image order) and differences element by element, and the time of few images."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J", [1, 2, 3, 8, 9, 24, 25, 48, 49, 96, 97, 113])
@pytest.mark.parametrize("m,n", [(1, 1), (5, 13), (8, 16), (33, 31)])
def test_values(J, m, n):
    from paper_1411_2860_amd import projgemm as pg
    rng = np.random.default_rng(J + m)
    X = (rng.standard_normal((J, m, n)) * 50).astype(np.float32)
    mean, out = pg.images_center(torch.from_numpy(X).cuda())
    total = np.zeros((m, n), np.float32)
    for x in X:                                             # FP32 sum in image order
        total += x
    want = (total.astype(np.float64) / J).astype(np.float32)
    got = mean.cpu().numpy()
    assert np.all(np.abs(got - want) <= 2.0 ** -23 * np.abs(want))       # division to 1 ulp
    assert np.array_equal(out.cpu().numpy(), X - got)
    sub = pg.images_subtract(torch.from_numpy(X).cuda(), mean)
    assert np.array_equal(sub.cpu().numpy(), X - got)


def _graph_us(fn, n=100):
    for _ in range(3):
        fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(n):
            fn()
    ts = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        ts.append(a.elapsed_time(b) * 1e3 / n)
    return float(np.median(ts))


def test_time_of_few_images():
    """One image of 288 x 288: centring moves the bytes of a subtraction (one array
    read, two written, against two and one), so it may take 1.5 times its time."""
    from paper_1411_2860_amd import projgemm as pg
    X = torch.randn((1, 288, 288), device="cuda")
    mean, out = X[0].clone(), torch.empty_like(X)
    center = _graph_us(lambda: pg.images_center(X, out=out))
    subtract = _graph_us(lambda: pg.images_subtract(X, mean, out=out))
    assert center <= 1.5 * subtract, (center, subtract)
