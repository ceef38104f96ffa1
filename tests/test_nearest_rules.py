"""CPU checks of how a large batch's nearest probes are scanned and bounded: the library's own header, compiled on the spot."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

SHIM = """
#include "ivfpq_nearest_rules.hpp"
extern "C" int wave_k() { return ivfpq::kBoundWaveK; }
extern "C" int shares() { return ivfpq::kBoundShares; }
extern "C" int room() { return ivfpq::kBoundCand; }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    where = tmp_path_factory.mktemp("rules")
    (where / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_06672_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, str(where / "shim.cpp"), "-o", str(where / "shim.so")], check=True)
    return ctypes.CDLL(str(where / "shim.so"))


def _let_in(key, k, shares):
    # values not above the k-th of the minima (its low 9 bits set)
    padded = np.full(-(-len(key) // shares) * shares, 0xFFFFFFFF, np.uint32)
    padded[:len(key)] = key
    upto = np.sort(padded.reshape(-1, shares).min(axis=0))[k - 1] | 0x1FF
    return int((key <= upto).sum())


@pytest.mark.parametrize("length", [128, 256, 300, 1_000, 4_000, 20_000])
def test_a_wave_has_room_for_what_the_first_bound_lets_in(rules, length):
    # values that do not cluster: always up to k = 100, in 9 lists of 10 at the largest k (500 lists: at 20,000 values 4 % +- 0.9 are expected)
    rng = np.random.default_rng(length)
    most = {100: 0, rules.wave_k(): 50}
    for _ in range(500):
        key = (rng.chisquare(32, length) * 10).astype(np.float32).view(np.uint32)
        for k in most:
            n = _let_in(key, k, rules.shares())
            assert n >= k
            most[k] -= n > rules.room()
    assert min(most.values()) >= 0
