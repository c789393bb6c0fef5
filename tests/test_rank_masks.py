"""The rank of a factor from elimination on its masks against elimination on
its entries: every shape, all densities, dependent rows; left open (-1) only
from order 3 on."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rank") / "rank_shim.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so,
                           os.path.join(HERE, "rank_shim.cpp")])
    lib = C.CDLL(so)
    for f in (lib.shim_rank_entries, lib.shim_rank_masks):
        f.argtypes = [C.c_uint64, C.c_uint64, C.c_int, C.c_int, C.c_int]
    return lib


SHAPES = sorted({(r, c) for r in range(1, 9) for c in range(1, 9)} | {(2, 32), (32, 2), (1, 64),
                                                                    (64, 1), (4, 16), (3, 21)})


@pytest.mark.parametrize("z2", [0, 1])
def test_masks_equal_entries(shim, z2):
    rng = np.random.default_rng(17 + z2)
    left_open = 0
    for rows, cols in SHAPES:
        for _ in range(400):
            M = rng.integers(-1, 2, (rows, cols)) * (rng.random((rows, cols)) < rng.random())
            if rows > 2 and rng.random() < 0.5:     # a dependent row
                a, b = rng.integers(0, rows, 2)
                M[a] = rng.choice([-1, 1]) * M[b]
            flat = M.reshape(-1)
            d = sum(1 << e for e in range(flat.size) if flat[e])
            s = 0 if z2 else sum(1 << e for e in range(flat.size) if flat[e] < 0)
            want = shim.shim_rank_entries(d, s, rows, cols, z2)
            got = shim.shim_rank_masks(d, s, rows, cols, z2)
            if got < 0:
                left_open += 1
                assert not z2 and want >= 3 and min(rows, cols) > 3, (rows, cols, M)
            else:
                assert got == want, (rows, cols, M)
    assert z2 or left_open > 0
