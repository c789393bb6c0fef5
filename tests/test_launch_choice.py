"""The library's choice of strategy and lanes, on the host."""
import ctypes as C
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("launch") / "launch_shim.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so,
                           os.path.join(HERE, "launch_shim.cpp")])
    return C.CDLL(so)


def rounds(walks, lanes, cap, max_len, indexed):
    """rounds of the resident wavefronts of 256 CUs: 160 KiB of LDS a CU in pieces of 1,280
    bytes, sixteen wavefronts at most"""
    entry = 16 if max_len > 32 else 4 if indexed and max_len <= 16 else 8
    rows = -(-cap // 4) * 4 if indexed else -(-cap // 2) * 2
    per_walk = rows * 3 * entry + (cap * 24 if indexed else 0)
    per_wave = 64 // lanes
    resident = min(16, 128 // -(-per_wave * per_walk // 1280))
    return -(-walks // (256 * resident * per_wave))


@pytest.mark.parametrize("max_len", [9, 16, 25, 32])
@pytest.mark.parametrize("objective", [0, 1])
def test_full_chips_take_no_round_more_than_needed(shim, max_len, objective):
    for cap in range(9, 97):
        for walks in range(8193, 66000, 511):
            strategy, lanes = divmod(shim.shim_default(cap, max_len, walks, objective), 100)
            if strategy == 2:
                continue
            assert lanes in (8, 16) and strategy == (3 if cap <= 64 else 1)
            other = 24 - lanes
            assert (rounds(walks, lanes, cap, max_len, cap <= 64) <=
                    rounds(walks, other, cap, max_len, cap <= 64)), (cap, walks, lanes)
