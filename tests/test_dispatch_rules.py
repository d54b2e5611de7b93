"""Rules that choose a kernel by size, called in the library without a GPU
(their C++ names): each figure beside a rule is a choice it has to make."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def rule():
    from paper_1411_2860_amd import projgemm as pg
    L = pg.lib()

    def get(name, res, *args):
        f = getattr(L, name)
        f.restype, f.argtypes = res, list(args)
        return f
    return get


F64, F32, BF16 = 0, 1, 2
SPLIT128, FP32_64 = 17, 5


@pytest.mark.parametrize("P,Q,nkb,cfg", [
    # an edge leaves a quarter or more of the 128 x 128 tiles' area empty
    (1, 20000, 32, FP32_64), (64, 20000, 8, FP32_64), (64, 20000, 96, FP32_64), (20000, 64, 96, FP32_64),
    (129, 8400, 96, FP32_64), (129, 17000, 2, FP32_64), (192, 17000, 32, FP32_64), (32, 70000, 32, FP32_64),
    # short contractions
    (1500, 1500, 1, FP32_64), (1500, 1500, 8, FP32_64), (1024, 2176, 4, FP32_64), (2000, 2100, 4, FP32_64),
    (4096, 4096, 1, FP32_64),
    # full tiles, long contractions
    (96, 17000, 32, SPLIT128), (1500, 1500, 32, SPLIT128), (1920, 1920, 8, SPLIT128), (2000, 2100, 32, SPLIT128),
    (193, 17000, 32, SPLIT128), (1024, 8192, 2, SPLIT128), (1024, 8192, 128, SPLIT128), (1003, 3001, 102, SPLIT128),
    # too few tiles
    (512, 2048, 128, FP32_64), (4096, 512, 512, FP32_64), (1274, 1561, 336, FP32_64), (1344, 1536, 16, FP32_64),
    (4100, 512, 384, SPLIT128)])
def test_fp32_tile(rule, P, Q, nkb, cfg):
    f = rule("_ZN2pj19gemm_default_configEilll", ctypes.c_int, ctypes.c_int, *[ctypes.c_long] * 3)
    assert f(F32, P, Q, nkb) == cfg


FULL, BLOCK = 0, 1


@pytest.mark.parametrize("blocks,L,r,rate,rows", [
    (8, 1, 1, FULL, 64), (32, 2, 1, BLOCK, 64), (40, 1, 1, FULL, 128), (40, 8, 4, FULL, 128), (49, 2, 1, BLOCK, 128),
    (100, 1, 1, FULL, 128), (128, 1, 1, BLOCK, 128), (160, 1, 1, FULL, 512), (160, 2, 1, BLOCK, 512),
    (160, 2, 1, FULL, 128), (160, 4, 1, BLOCK, 128), (160, 8, 8, FULL, 128), (250, 1, 1, FULL, 512),
    (250, 2, 2, FULL, 512), (250, 4, 4, FULL, 128), (250, 4, 4, BLOCK, 512), (250, 8, 1, FULL, 512),
    (257, 8, 8, FULL, 512), (8192, 2, 1, BLOCK, 512)])
def test_short_block_rows(rule, blocks, L, r, rate, rows):
    f = rule("_ZN2pj15corr_small_rowsEliii", ctypes.c_int, ctypes.c_long, *[ctypes.c_int] * 3)
    assert f(512 * blocks, L, r, rate) == rows


def test_short_block_rounds(rule):
    """No cut leaves a second round of 64-row workgroups or a third of 128-row
    ones (L = 1)."""
    f = rule("_ZN2pj15corr_small_rowsEliii", ctypes.c_int, ctypes.c_long, *[ctypes.c_int] * 3)
    for rows in range(1, 300 * 512, 97):
        cut = f(rows, 1, 1, FULL)
        assert cut == 512 or -(-rows // cut) <= (256 if cut == 64 else 512), rows


@pytest.mark.parametrize("prec,P,K,L,r,aligned,split,columns", [
    (F32, 4097, 4096, 32, 32, 0, 0, 1), (F32, 101, 8192, 256, 64, 0, 0, 1), (BF16, 257, 4096, 64, 64, 0, 0, 1),
    (F32, 4096, 4096, 8, 4, 1, 0, 1), (F32, 1000, 2048, 16, 16, 1, 0, 1), (F32, 4096, 4096, 64, 8, 1, 0, 1),
    (F32, 4096, 4096, 64, 16, 1, 0, 1), (F32, 4096, 4096, 64, 64, 1, 0, 0), (F32, 2048, 4096, 64, 8, 1, 0, 0),
    (F32, 256, 4096, 64, 8, 1, 0, 0), (F32, 1024, 1024, 64, 64, 1, 0, 0), (F32, 128, 8192, 64, 16, 1, 0, 0),
    (F32, 4096, 4096, 256, 16, 1, 0, 0), (F32, 4096, 4096, 256, 256, 1, 0, 0), (F32, 4096, 4096, 32, 32, 1, 0, 1),
    (F32, 1000, 2048, 32, 16, 1, 0, 0), (F32, 4096, 4096, 48, 20, 1, 0, 0), (F32, 64, 65536, 32, 8, 1, 0, 0),
    (BF16, 256, 4096, 64, 8, 1, 0, 1), (BF16, 256, 4096, 64, 16, 1, 0, 1), (BF16, 1024, 4096, 64, 32, 1, 0, 0),
    (BF16, 4096, 4096, 64, 64, 1, 0, 1),
    (BF16, 4096, 4096, 256, 16, 1, 0, 0), (BF16, 1024, 4096, 128, 16, 1, 0, 0), (F32, 1024, 4096, 32, 4, 1, 0, 1),
    (BF16, 192, 128, 64, 15, 1, 0, 0), (BF16, 192, 128, 64, 8, 1, 0, 1), (BF16, 576, 320, 48, 14, 1, 0, 0),
    (BF16, 512, 512, 32, 32, 1, 0, 0), (BF16, 3352, 363, 28, 19, 1, 0, 1), (BF16, 8064, 2224, 20, 18, 1, 0, 1),
    (BF16, 4096, 4096, 32, 32, 1, 0, 1),
    (F64, 1024, 1024, 64, 33, 1, 0, 1), (F64, 1024, 1024, 64, 64, 1, 0, 0), (F64, 2048, 2048, 64, 64, 1, 0, 1),
    (F64, 1024, 1024, 16, 4, 1, 1, 1), (F64, 1024, 1024, 32, 16, 1, 1, 0), (F64, 2048, 2048, 256, 200, 1, 1, 0),
    (F64, 1000, 2048, 64, 17, 1, 1, 1), (F32, 1024, 1024, 12, 5, 1, 1, 0), (F32, 4096, 4096, 12, 5, 1, 1, 1),
    (F32, 4096, 4096, 48, 6, 1, 1, 0)])
def test_pack_columns(rule, prec, P, K, L, r, aligned, split, columns):
    f = rule("_ZN2pj16pack_columns_payEilliiii", ctypes.c_bool, ctypes.c_int, *[ctypes.c_long] * 2, *[ctypes.c_int] * 4)
    assert f(prec, P, K, L, r, aligned, split) == bool(columns)


@pytest.mark.parametrize("prec,default", [("bf16", 16), ("bf16x3", 16), ("f16", 16), ("f32", 17), ("f64", 0), ("fp8", 0)])
@pytest.mark.parametrize("shapes,small", [
    ([(1024, 1024, 1024)] * 10, False), ([(1024, 1024, 1024)] * 10 + [(32, 32, 65536)], True),
    ([(700, 700, 700)] * 30 + [(60, 60, 60000)] * 4, True), ([(8, 4096, 4096)] * 8, True),
    ([(4096, 4096, 4096)] * 8 + [(100, 100, 2048)] * 9, False), ([(1500, 2500, 1000)] * 24 + [(32, 32, 4096)], False)])
def test_batch_configuration(prec, default, shapes, small):
    """The workspace, whose item table follows the tiles, tells which configuration a
    batch takes: 0 where its small tiles would outlast the large ones."""
    if prec == "f32" and shapes[0][0] == 8:               # large and small tiles have the same rows
        small = False
    from paper_1411_2860_amd import projgemm as pg
    descs = (pg.GemmDesc * len(shapes))(*[pg.GemmDesc(m, w, k, b"N", b"N", 256, k, 256, w, 256, w) for m, w, k in shapes])
    auto, chosen = (pg.gemm_batched_workspace_bytes(descs, 16, 4, prec, c) for c in (-1, 0 if small else default))
    assert auto == chosen > 0
    if default == 16 and shapes[0][0] > 8:                # FP32's two have tiles of one size
        assert pg.gemm_batched_workspace_bytes(descs, 16, 4, prec, default if small else 0) != auto


@pytest.mark.parametrize("f64,L,r,in_trans,out_trans,once", [
    (0, 16, 11, 0, 1, 1), (0, 10, 4, 0, 0, 1), (0, 17, 4, 0, 0, 0), (0, 20, 11, 0, 1, 0), (0, 20, 11, 0, 0, 1),
    (0, 64, 16, 1, 1, 1), (0, 64, 17, 1, 1, 0), (0, 64, 16, 1, 0, 0), (1, 8, 2, 0, 0, 0)])
def test_synthesis_reads_once(rule, f64, L, r, in_trans, out_trans, once):
    f = rule("_ZN2pj11expand_onceEiiiii", ctypes.c_bool, *[ctypes.c_int] * 5)
    assert f(f64, L, r, in_trans, out_trans) == bool(once)
