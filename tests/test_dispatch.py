"""Host-side rules that choose how a launch is cut, called in the built library by their C++ names. No GPU needed."""
import ctypes as C
import os
import random
import time

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2506_15733_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return binding.load_library()


class DecodeRuns(C.Structure):
    _fields_ = [("tiles", C.c_int32), ("count", C.c_int32)]


def decode_runs(lib, lens, units, per_split, part_floats):
    f = lib._Z16plan_decode_runsPKiiilmm
    f.restype = DecodeRuns
    f.argtypes = [C.POINTER(C.c_int32), C.c_int, C.c_int, C.c_long, C.c_size_t, C.c_size_t]
    r = f((C.c_int32 * len(lens))(*lens), len(lens), -1, units, per_split, part_floats)
    return r.tiles, r.count


def decode_runs_by_definition(lens, units, per_split, part_floats):
    tiles = [-(-n // 64) for n in lens]
    longest = max(max(tiles), 1)
    run = max(-(-longest // 32), min(sum(tiles) * units // 512, longest))
    while run < longest and (sum(-(-t // run) for t in tiles) * units > 512 or -(-longest // run) * per_split > part_floats):
        run += 1
    return run, -(-longest // run)


def test_runs_of_generation_attention_are_the_shortest_that_fit(lib):
    rng = random.Random(3)
    for _ in range(300):
        lens = [int(2 ** rng.uniform(0, 14)) for _ in range(rng.choice((1, 2, 3, 17, 64, 300)))]
        units = rng.choice((1, 2, 4, 9, 64, 513))
        per_split = rng.randint(1, 1 << 20)
        args = lens, units, per_split, rng.choice((0, per_split, 3 * per_split, 1 << 40))
        assert decode_runs(lib, *args) == decode_runs_by_definition(*args), args
    assert decode_runs(lib, [0], 1, 1, 100) == (1, 1)


def test_runs_are_found_quickly_where_no_length_fits(lib):
    """256 beams, one of them long, and more workgroups than are resident: a search through all run lengths takes about
    half a million divisions, a bisection a few thousand. The bound lies an order of magnitude from both."""
    lens = [1024] * 255 + [131072]
    best = min(_timed(lambda: decode_runs(lib, lens, 4, 1, 1 << 40)) for _ in range(20))
    assert decode_runs(lib, lens, 4, 1, 1 << 40) == (2048, 1)
    assert best < 3e-4, best


def _timed(f):
    t = time.perf_counter()
    f()
    return time.perf_counter() - t
