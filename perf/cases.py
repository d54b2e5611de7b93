"""Performance cases of the projected GEMM / cross-correlation library.

Each case is one call (or one training step of one layer) through the public
Python entry points, on inputs of the kind that bench.py and the tests use:
smoothed-noise images with values 0..255, smoothed sequences, Gaussian
matrices and AR(2) signals, made here on the GPU from the seed alone.

  listed()            the fixed cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) inputs, basis and packed database that a program holds
  run(state)          one pass; returns the outputs whole
  work(case)          bytes and flops that the pass cannot do without
  exact(case, seed)   the projected result in FP64, from torch alone
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1411_2860_amd import projgemm as pg
from paper_1411_2860_amd.autograd import proj_matmul

DEV = "cuda"

LISTED = [
    # Smallest calls: the FP64 parity configuration of the tests and of
    # bench.py (256^3, L = 16), bound by launches and latency.
    dict(name="gemm_f64_256", kind="gemm", M=256, W=256, K=256, L=16, r=4, basis="dct2", prec="f64", transA=False,
         transB=False),
    # The headline: 1024 query images of 64 x 64 against 8192 database images
    # stored as rows, 16 of 64 DCT projections, FP32.
    dict(name="recognition_f32_r16", kind="gemm", M=1024, W=8192, K=4096, L=64, r=16, basis="dct2", prec="f32",
         transA=False, transB=True),
    # An ordinary product with odd sizes: rows not 16-byte aligned, the last
    # group and the last tiles partly empty.
    dict(name="gemm_f32_ragged", kind="gemm", M=1003, W=3001, K=2101, L=16, r=6, basis="haar", prec="f32",
         transA=False, transB=False),
    # Serving: the database is packed once, each call projects the queries
    # and contracts.
    dict(name="static_db_bf16_r16", kind="static", M=1024, W=8192, K=4096, L=64, r=16, rmax=64, basis="dct2",
         prec="bf16"),
    # The cheapest end of the precision ladder on the recognition shape.
    dict(name="recognition_fp8_r8", kind="gemm", M=1024, W=8192, K=4096, L=64, r=8, basis="dct2", prec="fp8",
         transA=False, transB=True),
    # One linear layer of a training step, forward and backward.
    dict(name="linear_bf16_r8_fwd_bwd", kind="linear", M=4096, W=4096, K=4096, L=64, r=8, basis="dct2", prec="bf16"),
    # Many uneven problems in one call (sides 128..4096).
    dict(name="batched_bf16x3_24", kind="batched", count=24, lo=128, hi=4096, shapes=64, L=16, r=4, basis="dct2",
         prec="bf16x3"),
    # 2D-PCA training: centring and the image scatter matrix of 75 images of
    # 288 x 288 (a skinny output, a long contraction, the left side transposed).
    dict(name="pca2d_scatter_f32", kind="scatter", J=75, m=288, n=288, L=8, r=1, basis="dct2", prec="f32"),
    # Template search, every lag: 2^22 samples, 4096-sample template, 16 of
    # 256 projections.
    dict(name="conv_full_l256_r16", kind="conv", W=1 << 22, N=4096, L=256, r=16, basis="dct2", rate="full",
         mode="xcorr"),
    # The same at the block rate (aligned lags computed, the rest
    # interpolated), long template.
    dict(name="conv_block_l256_r16", kind="conv", W=1 << 22, N=16384, L=256, r=16, basis="dct2", rate="block",
         mode="xcorr"),
    # The paper's operating point: one of two Haar projections, half of the
    # samples, a block of 20000 samples; bound by launches and latency.
    dict(name="conv_point_20000", kind="conv", W=20000, N=600, L=2, r=1, basis="haar", rate="block", mode="xcorr"),
    # Long template, short blocks, all projections: the frequency domain.
    dict(name="conv_long_l16_r16", kind="conv", W=1 << 22, N=16384, L=16, r=16, basis="dct2", rate="full",
         mode="conv"),
]


def listed():
    return [dict(c) for c in LISTED]


# ------------------------------------------------------------------- drawing

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    """A size spread over the logarithm of its range: a third multiples of
    64, a third of 8, a third as drawn (mostly odd)."""
    n = _log(rng, lo, hi)
    q = rng.choice((64, 8, 1))
    return max(lo, n // q * q)


def _basis(rng, L):
    return rng.choice(("dct2", "haar")) if L & (L - 1) == 0 else "dct2"


def draw(rng):
    kind = rng.choice(("gemm", "gemm", "gemm", "static", "linear", "batched", "scatter", "conv", "conv", "conv"))
    if kind in ("gemm", "static"):
        L = rng.choice((8, 12, 16, 32, 64))
        prec = rng.choice(("f32", "f32", "bf16", "bf16x3", "f16", "f16x3", "fp8", "f64"))
        r = min(L, _log(rng, 1, L))
        if prec == "fp8":
            r = min(r, 8)
        hi = 512 if prec == "f64" else 8192
        c = dict(kind=kind, M=_side(rng, 64, hi // 4), W=_side(rng, 64, hi), K=_side(rng, 128, hi // 2), L=L, r=r,
                 basis=_basis(rng, L), prec=prec)
        if kind == "static":
            return dict(c, rmax=min(L, max(r, 8 if prec == "fp8" else 16)))
        return dict(c, transA=rng.random() < 0.2, transB=rng.random() < 0.5)
    if kind == "linear":
        L = rng.choice((8, 16, 64))
        return dict(kind=kind, M=_side(rng, 256, 4096), W=_side(rng, 256, 4096), K=_side(rng, 256, 4096), L=L,
                    r=min(L, _log(rng, 1, 16)), basis=_basis(rng, L), prec=rng.choice(("bf16", "bf16", "f16", "f32")))
    if kind == "batched":
        L = rng.choice((8, 16, 64))
        return dict(kind=kind, count=rng.randint(4, 20), lo=128, hi=_side(rng, 512, 4096),
                    shapes=rng.randint(0, 1 << 20), L=L, r=min(L, _log(rng, 1, 8)), basis=_basis(rng, L),
                    prec=rng.choice(("bf16x3", "bf16", "f32", "fp8")))
    if kind == "scatter":
        m = _side(rng, 64, 288)
        L = rng.choice((8, 12, 16))
        return dict(kind=kind, J=rng.randint(10, 75), m=m, n=_side(rng, 64, 288), L=L, r=rng.randint(1, L // 2),
                    basis="dct2", prec="f32")
    rate = rng.choice(("full", "full", "block"))
    L = rng.choice((2, 4, 8, 16, 32, 64, 128, 256))
    W = _side(rng, 20000, 1 << 22)
    N = min(W // 4, _side(rng, 256, 16384))
    r = min(L, _log(rng, 1, L))
    while rate == "full" and 2.0 * W * r * (N / L + 1) > 4e10 and L >= 16 and r > 1:
        r //= 2
    return dict(kind=kind, W=W, N=N, L=L, r=r, basis=_basis(rng, L), rate=rate,
                mode=rng.choice(("xcorr", "conv")))


# -------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1411 * 1000003 + int(seed))
    return g


def _band(n, sigma=4.0):
    """n x (n + 2 rad) matrix of a valid Gaussian smoothing."""
    rad = int(math.ceil(4.0 * sigma))
    x = torch.arange(-rad, rad + 1, dtype=torch.float32, device=DEV)
    w = torch.exp(-0.5 * (x / sigma) ** 2)
    w = w / w.sum()
    B = torch.zeros((n, n + 2 * rad), dtype=torch.float32, device=DEV)
    i = torch.arange(n, device=DEV)
    for t in range(2 * rad + 1):
        B[i, i + t] = w[t]
    return B


def _to_bytes(z):
    lo, hi = z.min(dim=1, keepdim=True).values, z.max(dim=1, keepdim=True).values
    return torch.round((z - lo) / (hi - lo) * 255.0)


def _sequences(n, length, g):
    """n smoothed noise sequences with values 0..255, one a row."""
    B = _band(length)
    return _to_bytes(torch.randn((n, B.shape[1]), generator=g, device=DEV) @ B.t().contiguous())


def _images(n, side_m, side_n, g):
    """n smoothed noise images with values 0..255, one a row."""
    Bm, Bn = _band(side_m), _band(side_n)
    z = torch.randn((n, Bm.shape[1], Bn.shape[1]), generator=g, device=DEV)
    z = (z.reshape(-1, Bn.shape[1]) @ Bn.t().contiguous()).reshape(n, Bm.shape[1], side_n)
    z = z.transpose(1, 2).contiguous().reshape(-1, Bm.shape[1]) @ Bm.t().contiguous()
    return _to_bytes(z.reshape(n, side_n * side_m))


def _rows(n, K, g):
    return _images(n, 64, 64, g) if K == 4096 else _sequences(n, K, g)


def _signal(n, g):
    """AR(2) process with poles 0.95 and 0.9 (its impulse response, 1024 taps)."""
    e = torch.randn(n + 1024, generator=g, device=DEV, dtype=torch.float64)
    t = torch.arange(1024, device=DEV, dtype=torch.float64)
    h = (0.95 ** (t + 1) - 0.9 ** (t + 1)) / 0.05
    F = 1 << (n + 2048).bit_length()
    s = torch.fft.irfft(torch.fft.rfft(e, F) * torch.fft.rfft(h, F), F)
    return s[1024:1024 + n].float().contiguous()


def _shapes(case):
    rng = np.random.default_rng(case["shapes"])
    return [tuple(int(v) for v in rng.integers(case["lo"], case["hi"] + 1, size=3)) for _ in range(case["count"])]


def _inputs(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    dt = torch.float64 if case.get("prec") == "f64" else torch.float32
    if kind in ("gemm", "static"):
        M, W, K = case["M"], case["W"], case["K"]
        A = _rows(M, K, g).to(dt)
        if kind == "static" or case["transB"]:
            B = _rows(W, K, g).to(dt)                                        # database images, W x K
        else:
            B = torch.randn((K, W), generator=g, device=DEV, dtype=torch.float32).to(dt)
        return dict(A=A.t().contiguous() if case.get("transA") else A, B=B)
    if kind == "linear":
        M, W, K = case["M"], case["W"], case["K"]
        return dict(X=_rows(M, K, g) / 255.0, Wt=torch.randn((K, W), generator=g, device=DEV) / math.sqrt(K),
                    dY=torch.randn((M, W), generator=g, device=DEV) / M)
    if kind == "batched":
        As = [_sequences(m, k, g) for m, w, k in _shapes(case)]
        return dict(As=As, Bs=[torch.randn((k, w), generator=g, device=DEV) for m, w, k in _shapes(case)])
    if kind == "scatter":
        return dict(X=_images(case["J"], case["n"], case["m"], g).reshape(case["J"], case["m"], case["n"]))
    s = _signal(case["W"], g)
    o = int(np.random.default_rng(seed).integers(0, case["W"] - case["N"] + 1))
    return dict(s=s, k=s[o:o + case["N"]].clone())


def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"] = dict(case)
    st["basis"] = pg.Basis(case["basis"], case["L"])
    if case["kind"] == "static":       # the database, packed once
        st["db"] = pg.pack_b(st.pop("B"), case["rmax"], st["basis"], prec=case["prec"], transB=True)
    if case["kind"] == "linear":
        st["X"].requires_grad_()
        st["Wt"].requires_grad_()
    return st


# ---------------------------------------------------------------------- runs

def run(st):
    c, b = st["case"], st["basis"]
    kind = c["kind"]
    if kind == "gemm":
        return pg.gemm(st["A"], st["B"], c["r"], b, prec=c["prec"], transA=c["transA"], transB=c["transB"])
    if kind == "static":
        Ap = pg.pack_a(st["A"], c["r"], b, prec=c["prec"])
        return pg.gemm_packed(Ap, st["db"], c["r"], c["M"], c["W"], c["K"], c["L"], c["r"], c["rmax"],
                              prec=c["prec"])
    if kind == "linear":
        Y = proj_matmul(st["X"], st["Wt"], c["r"], b, c["prec"])
        dX, dW = torch.autograd.grad(Y, (st["X"], st["Wt"]), st["dY"])
        return Y.detach(), dX, dW
    if kind == "batched":
        return pg.gemm_batched(st["As"], st["Bs"], c["r"], b, prec=c["prec"])
    if kind == "scatter":
        mean, X = pg.images_center(st["X"])
        A = X.reshape(c["J"] * c["m"], c["n"])
        return mean, pg.symmetrize(pg.gemm(A, A, c["r"], b, prec=c["prec"], transA=True))
    return pg.conv1d(st["s"], st["k"], c["r"], b, mode=c["mode"], rate=c["rate"])


# ----------------------------------------------------------------- work

def _gemm_work(M, W, K, L, r, e=4):
    """Operands read and result written once; the projections of both sides
    and the contraction over r projections."""
    G = -(-K // L)
    return e * (M * K + K * W + M * W), 2.0 * M * W * r * G + 2.0 * (M + W) * K * r


def work(case):
    c, kind = case, case["kind"]
    if kind == "gemm":
        b, f = _gemm_work(c["M"], c["W"], c["K"], c["L"], c["r"], 8 if c["prec"] == "f64" else 4)
    elif kind == "static":
        size = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2, "bf16x3": 4, "f16x3": 4, "fp8": 1}[c["prec"]]
        e, G = 8 if c["prec"] == "f64" else 4, -(-c["K"] // c["L"])
        b = e * (c["M"] * c["K"] + c["M"] * c["W"]) + size * c["W"] * G * c["r"]
        f = 2.0 * c["M"] * c["W"] * c["r"] * G + 2.0 * c["M"] * c["K"] * c["r"]
    elif kind == "linear":
        M, W, K, r = c["M"], c["W"], c["K"], c["r"]
        G = -(-K // c["L"])
        b = 4 * 2 * (M * K + K * W + M * W)
        f = 3 * 2.0 * M * W * r * G + 4.0 * (M + W) * K * r
    elif kind == "batched":
        ws = [_gemm_work(m, w, k, c["L"], c["r"]) for m, w, k in _shapes(c)]
        b, f = sum(x[0] for x in ws), sum(x[1] for x in ws)
    elif kind == "scatter":
        K, n = c["J"] * c["m"], c["n"]
        b = 4 * (K * n + c["m"] * n + n * n)
        f = 2.0 * n * n * c["r"] * -(-K // c["L"]) + 4.0 * n * K * c["r"]
    else:
        W, N, L, r = c["W"], c["N"], c["L"], c["r"]
        nout, taps = W - N + 1, -(-N // L)
        b = 4 * (W + N + nout)
        if c["rate"] == "block":
            f = 2.0 * (nout / L) * r * taps
        else:      # direct sums, or transforms of the projected rows
            f = min(2.0 * nout * r * taps, 5.0 * (r + L) * (W / L) * math.log2(max(4 * taps, 2)) +
                    8.0 * r * L * (W / L))
        f += 2.0 * (W + N) * r
    return {"bytes": float(b), "flops": float(f)}


# ----------------------------------------------------------------- FP64 values

def _matrix(kind, L):
    """Orthonormal L x L basis (columns = projections, DCT-II by frequency,
    Haar from the coarsest scale), FP64."""
    C = np.zeros((L, L))
    if kind == "dct2":
        t = np.arange(L)
        for l in range(L):
            C[:, l] = math.sqrt((1.0 if l == 0 else 2.0) / L) * np.cos(math.pi * (t + 0.5) * l / L)
    else:
        C[:, 0] = 1.0 / math.sqrt(L)
        l, n = 1, L
        while n > 1:                       # wavelets of support n
            for sft in range(L // n):
                C[sft * n:sft * n + n // 2, l] = 1.0 / math.sqrt(n)
                C[sft * n + n // 2:(sft + 1) * n, l] = -1.0 / math.sqrt(n)
                l += 1
            n //= 2
    return torch.from_numpy(C).to(DEV)


def _project(X, C, r):
    """First r projections of the aligned groups of every row: rows x (G r)."""
    L = C.shape[0]
    rows, K = X.shape
    G = -(-K // L)
    Z = torch.zeros((rows, G * L), dtype=torch.float64, device=X.device)
    Z[:, :K] = X
    return (Z.reshape(rows * G, L) @ C[:, :r].contiguous()).reshape(rows, G * r)


def _spread(H, C, r, K):
    """Transpose of _project: rows x K."""
    L = C.shape[0]
    rows = H.shape[0]
    return (H.reshape(-1, r) @ C[:, :r].t().contiguous()).reshape(rows, -1)[:, :K].contiguous()


def _conv_exact(case, s, k, C):
    W, N, L, r = case["W"], case["N"], case["L"], case["r"]
    s, k = s.double(), k.double()
    if case["mode"] == "conv":
        k = torch.flip(k, (0,))
    st = _spread(_project(s[None], C, r), C, r, -(-W // L) * L)[0]
    st = torch.cat([st, st.new_zeros(L)])
    F = 1 << (W + L).bit_length()
    y = torch.fft.irfft(torch.fft.rfft(st, F) * torch.fft.rfft(k, F).conj(), F)[:W - N + 1]
    if case["rate"] == "full":
        return y.contiguous()
    m = torch.arange(W - N + 1, device=DEV)
    a, top = m // L, (W - N) // L
    lo, hi = y[a * L], y[torch.clamp(a + 1, max=top) * L]
    return lo + (m % L).double() / L * (hi - lo)


def exact(case, seed):
    x = _inputs(case, seed)
    c, kind = case, case["kind"]
    C, r = _matrix(c["basis"], c["L"]), c["r"]
    if kind in ("gemm", "static"):
        A = x["A"].t() if c.get("transA") else x["A"]
        B = x["B"] if kind == "static" or c["transB"] else x["B"].t()
        return _project(A.double(), C, r) @ _project(B.double(), C, r).t().contiguous()
    if kind == "linear":
        X, Wt, dY = (x[n].double() for n in ("X", "Wt", "dY"))
        Xh, Wh = _project(X, C, r), _project(Wt.t(), C, r)
        K = X.shape[1]
        dX = _spread(dY @ Wh, C, r, K)
        dW = _spread(dY.t().contiguous() @ Xh, C, r, K).t().contiguous()
        return Xh @ Wh.t().contiguous(), dX, dW
    if kind == "batched":
        return [_project(A.double(), C, r) @ _project(B.double().t(), C, r).t().contiguous()
                for A, B in zip(x["As"], x["Bs"])]
    if kind == "scatter":
        X = x["X"].double()
        mean = X.mean(dim=0)
        A = _project((X - mean).reshape(-1, X.shape[2]).t().contiguous(), C, r)
        return mean, A @ A.t().contiguous()
    return _conv_exact(c, x["s"], x["k"], C)
