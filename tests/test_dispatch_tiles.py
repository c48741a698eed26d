"""The tile that a bf16 product is launched in, against the plan it refines. No GPU needed."""
import ctypes as C
import random

import pytest

from host_rules import BatchGeom, library

PLAN = ("256x256", "128x256", "128x128", "64x128", "32x128", "64x64", "32x64", "192x256", "64x128 short")


def plan(M, N, K, max_split, wide):
    f = library()._Z14mfma_gemm_planiiiibPiS_
    f.restype, f.argtypes = None, [C.c_int] * 4 + [C.c_bool] + [C.POINTER(C.c_int)] * 2
    tile, split = C.c_int(), C.c_int()
    f(M, N, K, max_split, wide, tile, split)
    return PLAN[tile.value], split.value


def launched(M, N, K, max_split=1, wide=False, beside=False):
    f = library()._Z14mfma_gemm_tileiiiibbPiS_
    f.restype, f.argtypes = None, [C.c_int] * 4 + [C.c_bool] * 2 + [C.POINTER(C.c_int)] * 2
    tile, split = C.c_int(), C.c_int()
    f(M, N, K, max_split, wide, beside, tile, split)
    return PLAN[tile.value], split.value


def test_slices_are_always_those_of_the_plan():
    """All tiles add a slice's products in the same order: with the plan's slices a product keeps its bits whichever tile it gets."""
    rng = random.Random(3)
    refined = set()
    for _ in range(20000):
        M = int(2 ** rng.uniform(0, 14.2))
        N, K = 64 * rng.randint(1, 700) + rng.choice((0, 0, 8, 3)), 64 * int(2 ** rng.uniform(0, 8.3))
        most, wide, beside = rng.choice((1, 2, 7, 16)), rng.random() < 0.2, rng.random() < 0.5
        before, after = plan(M, N, K, most, wide), launched(M, N, K, most, wide, beside)
        assert before[1] == after[1]
        if before[0] != after[0]:
            refined.add((before[0], after[0]))
            assert wide is False or after[0] == "192x256"
            assert beside or after[0] != "64x128 short"
    assert refined == {("256x256", "192x256"), ("128x256", "192x256"), ("64x128", "64x64"), ("64x128", "32x64"),
                       ("64x128", "64x128 short")}


@pytest.mark.parametrize("tile,max_split,M,N,K", [
    ("192x256", 1, 1100, 9728, 896), ("192x256", 1, 555, 37888, 3584), ("192x256", 16, 1600, 3584, 18944),
    ("256x256", 1, 1600, 17920, 1536), ("256x256", 1, 1600, 37888, 3584), ("256x256", 1, 2048, 37888, 3584),
    ("128x256", 1, 1600, 4608, 3584), ("128x256", 1, 1100, 4608, 3584),
    ("32x64", 1, 256, 2048, 1024), ("32x64", 1, 256, 2048, 1536),
    ("64x64", 16, 256, 1024, 1024),                  # 4 slices: 256 workgroups of 64 x 64
    ("64x64", 1, 555, 2048, 1536),                   # 288 workgroups, few weights
    ("64x64", 1, 650, 1536, 1536), ("64x64", 1, 768, 1536, 1536), ("64x64", 1, 900, 1152, 896), ("64x64", 1, 1152, 1024, 1024),
    ("64x128", 1, 256, 4608, 3584),                  # 288, and many
    ("64x128", 1, 320, 3584, 1024), ("64x128", 1, 256, 4608, 896),
    ("64x128", 1, 256, 5632, 1024), ("64x128", 1, 1024, 2048, 1536)])
def test_tiles_of_measured_products(tile, max_split, M, N, K):
    assert launched(M, N, K, max_split)[0] == tile


@pytest.mark.parametrize("tile,max_split,M,N,K", [
    ("64x128 short", 1, 256, 5632, 1024), ("64x128 short", 1, 1024, 2048, 1536),
    ("64x128", 1, 256, 4608, 3584),                  # 56 K-tiles
    ("64x128", 16, 256, 1536, 8960),                 # 28 K-tiles a slice
    ("64x64", 1, 40, 16384, 1024)])                  # few enough for the finer tiles
def test_rings_of_launches_beside_others(tile, max_split, M, N, K):
    assert launched(M, N, K, max_split, beside=True)[0] == tile


def test_only_the_caller_says_that_others_run_beside():
    f = library()._Z15launches_besidebRK9BatchGeom
    f.restype, f.argtypes = C.c_bool, [C.c_bool, C.POINTER(BatchGeom)]
    assert f(True, BatchGeom(B=1, n=8, L=32)) and not f(False, BatchGeom(B=1, n=8, L=32))
    assert not f(True, BatchGeom(B=1, n=1, L=2048)) and not f(True, BatchGeom(B=4, n=8, L=1))


def test_rotary_embedding_of_single_positions():
    """In the product where the plan wants no slices, the walk through K is short, or many small tiles share it."""
    f = library()._Z17qkv_rope_positioniiii
    f.restype, f.argtypes = C.c_bool, [C.c_int] * 4
    assert f(256, 2048, 1536, 16) and f(48, 4608, 3584, 16) and not f(128, 4608, 3584, 16)
    assert all(f(M, N, K, 1) for M in (33, 64, 256) for N in (2048, 4608) for K in (1024, 3584))
