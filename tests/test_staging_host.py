"""Host-only checks of the arithmetic that a launch shape's staging is derived with (csrc/sc_staging.h), compiled here for the CPU."""
import ctypes
import itertools
import os
import random
import subprocess

import pytest

import gpu_util as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def staging(tmp_path_factory):
    d = tmp_path_factory.mktemp("staging")
    src = d / "staging.cpp"
    src.write_text(
        '#include "sc_staging.h"\n'
        'extern "C" long long least(long long H, long long Hs, long long step, long long pad, long long tiles)\n'
        '{ return sc::least_staged_rows(H, Hs, step, pad, tiles); }\n'
        'extern "C" int columns(int widest, int block, int column, long long groups, long long threads, long long rows, long long run, long long minrun)\n'
        '{ return sc::load_columns(widest, block, column, groups, threads, rows, run, minrun); }\n')
    so = d / "staging.so"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                           "-I", os.path.join(ROOT, "paper_2112_15445_amd", "csrc"), str(src), "-o", str(so)])
    lib = ctypes.CDLL(str(so))
    lib.least.argtypes = [ctypes.c_longlong] * 5
    lib.least.restype = ctypes.c_longlong
    lib.columns.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong] * 5
    return lib


def _least(H, Hs, step, pad, tiles):
    rows = [min(Hs, H - r) - max(0, -r) for r in (t * step - pad for t in range(tiles))]
    return min((r for r in rows if r > 0), default=0)


def test_shortest_tile_is_the_first_or_the_last(staging):
    """Against the count over all tiles: filters, strides, paddings of more than a tile, tiles past the input."""
    for H, R, s, pad, TP in itertools.product((1, 2, 5, 9), (1, 2, 3, 5), (1, 2, 3), range(0, 8), (1, 2, 3, 7)):
        P = (H + 2 * pad - R) // s + 1
        if H + 2 * pad < R:
            continue
        TP = min(TP, P)
        args = (H, (TP - 1) * s + R, TP * s, pad, (P + TP - 1) // TP)
        assert staging.least(*args) == _least(*args), args
    rng = random.Random(1)
    for _ in range(3000):
        args = (rng.randint(1, 300), rng.randint(1, 40), rng.randint(1, 60), rng.randint(0, 90), rng.randint(1, 60))
        assert staging.least(*args) == _least(*args), args
    # (a tall layer, tiles of one row: no walk over them)
    assert staging.least(1 << 30, 1, 1, 0, 1 << 30) == 1


def test_columns_of_a_load_fit_the_shortest_run(staging):
    """The rule of both forms against the one written out in Python."""
    rng = random.Random(2)
    for _ in range(4000):
        widest, block, column = rng.choice([(2, 40, 64), (3, 32, 8), (3, 40, 12)])
        groups, threads = rng.randint(1, 300), rng.choice([256, 512])
        rows, run = rng.randint(1, 40), rng.randint(0, 200)
        minrun = rng.randint(0, run)
        got = staging.columns(widest, block, column, groups, threads, rows, run, minrun)
        assert 1 << got == G.load_columns(widest, block, column, groups, threads, rows, run, minrun), (groups, threads, rows, run, minrun)
        assert got == 0 or 1 << got <= minrun
