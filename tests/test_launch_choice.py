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


def test_autotuner_times_the_default(shim):
    """every launch once, and the one that a call without tuning takes among them"""
    out = (C.c_int * 64)()
    for cap in (1, 12, 35, 41, 49, 64, 65, 72, 88, 96, 97, 128, 129, 512):
        for walks in (1, 256, 1024, 3073, 4096, 4097, 8192, 8193, 18432, 65536):
            for max_len in (9, 32, 64):
                for objective in (0, 1):
                    n = shim.shim_candidates(cap, max_len, walks, objective, out, 64)
                    got = list(out[:n])
                    assert len(set(got)) == n <= 64
                    strategy, lanes = divmod(shim.shim_default(cap, max_len, walks, objective), 100)
                    for waves in (1, 2, 4):
                        assert 1000 * strategy + 10 * lanes + waves in got


def test_tuned_launch_serves_its_kind_of_batch_alone(shim):
    def serves(a, b):
        return shim.shim_serves((C.c_int * 5)(*a), (C.c_int * 5)(*b))
    tuned = [88, 20, 20480, 0, 0]      # capacity, max_len, walks, objective, mode
    assert serves(tuned, tuned) and serves(tuned, [88, 20, 17000, 0, 0])
    for k, other in enumerate((87, 16, 32768, 1, 1)):
        assert not serves(tuned, tuned[:k] + [other] + tuned[k + 1:])


def test_checked_walks_take_the_shape_of_unchecked_ones(shim):
    shapes = set()
    for cap in (12, 35, 41, 49, 64, 65, 72, 88, 96, 97, 128, 129, 512):
        for walks in (1, 1024, 3073, 4097, 8193, 18432, 65536):
            for max_len in (9, 32, 64):
                for objective in (0, 1):
                    for waves in (0, 4):
                        call = (cap, max_len, walks, objective, 0, 0, waves)
                        shapes.add(shim.shim_shape(*call, 0))
                        assert shim.shim_shape(*call, 1) == shim.shim_shape(*call, 0) > 0
                    # named: one shape a strategy, or refused
                    for strategy in (0, 1, 2, 3):
                        for lanes in (0, 4, 8, 16, 32, 64):
                            if strategy == lanes == 0:
                                continue
                            plain = shim.shim_shape(cap, max_len, walks, objective, strategy,
                                                    lanes, 1, 0)
                            check = shim.shim_shape(cap, max_len, walks, objective, strategy,
                                                    lanes, 1, 1)
                            one = plain > 0 and plain // 10 % 100 == (64 if plain // 1000 == 2
                                                                      else 8)
                            assert check == (plain if one or plain < 0 else -1)
    assert {s // 10 for s in shapes} >= {264, 332, 316, 308, 116, 108}
