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
extern "C" int by_groups(long long nq, int k, long long n, double mean, double typical, double longest, int bits, int pq_dim, int elem_bytes, int pairs, int eight) {
    return ivfpq::nearest_by_groups({nq, k, n, mean, typical, longest, bits, pq_dim, elem_bytes, pairs, eight != 0});
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    where = tmp_path_factory.mktemp("rules")
    (where / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_06672_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, str(where / "shim.cpp"), "-o", str(where / "shim.so")], check=True)
    lib = ctypes.CDLL(str(where / "shim.so"))
    lib.by_groups.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong] + [ctypes.c_double] * 3 + [ctypes.c_int] * 5
    return lib


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


def _by_groups(rules, nq, lists, length, bits, sub, elem, pairs, eight, k=10, typical=None, longest=None):
    return bool(rules.by_groups(nq, k, lists * length, length, typical or length, longest or length, bits, sub, elem, pairs, eight))


E5M3_64, HALF_32, E5M3_48, HALF_64X7 = (8, 64, 1, 4, True), (8, 32, 2, 4, True), (8, 48, 1, 2, False), (7, 64, 2, 2, False)
HALF_64X4, FLOAT_64X4, E5M3_64X4 = (4, 64, 2, 4, False), (4, 64, 4, 4, False), (4, 64, 1, 4, False)


@pytest.mark.parametrize("encoding,shape,groups", [
    # the measured side, where one of the two takes a tenth less of the nearest probes
    (HALF_64X4, (3_000, 500, 2_000), False), (HALF_64X4, (4_500, 2_000, 2_000), False), (HALF_64X4, (10_000, 500, 2_000), True),
    (HALF_64X4, (16_000, 1_000, 500), True), (FLOAT_64X4, (5_000, 2_000, 300), False), (FLOAT_64X4, (10_000, 1_000, 1_000), True),
    (E5M3_64X4, (10_000, 100, 8_000), False), (E5M3_64X4, (4_500, 500, 2_000), False), ((4, 32, 4, 4, False), (16_000, 500, 2_000), False),
    ((4, 32, 1, 4, False), (10_000, 1_000, 1_000), False), ((7, 32, 2, 2, False), (10_000, 64, 16_000), False),
    ((6, 64, 2, 2, False), (6_500, 2_000, 2_000), False), (HALF_64X7, (3_000, 1_000, 1_000), False), (HALF_64X7, (10_000, 500, 2_000), True),
    (E5M3_48, (3_000, 1_000, 1_000), False), (E5M3_48, (6_500, 500, 2_000), True), (E5M3_64, (4_500, 4_000, 250), False),
    (E5M3_64, (3_000, 1_000, 1_000), False), (E5M3_64, (10_000, 1_000, 1_000), True), (E5M3_64, (10_000, 2_000, 2_000), True),
    (HALF_32, (3_000, 250, 4_000), True), (HALF_32, (3_000, 3_000, 1_000), False)])
def test_nearest_probes_take_the_measured_side(rules, encoding, shape, groups):
    assert _by_groups(rules, *shape, *encoding) == groups


def test_one_long_list_keeps_a_workgroup_a_query(rules):
    # 10,000 queries, lists of 1,000 and one longer: 64 codes of 7 bits, four waves, up to 77 % slower in groups from 32 lengths on; 64 codes, eight
    # waves, faster at 32
    for lengths, four, eight in ((8, True, True), (13, True, True), (32, False, True), (64, False, False), (134, False, False)):
        typical = (1023 * 1000 ** 2 + (lengths * 1000) ** 2) / (1023 * 1000 + lengths * 1000)
        more = dict(typical=typical, longest=lengths * 1000)
        assert _by_groups(rules, 10_000, 1_024, 1_000, 7, 64, 1, 4, False, **more) == four
        assert _by_groups(rules, 10_000, 1_024, 1_000, *E5M3_64, **more) == eight


def test_what_takes_no_groups(rules):
    assert _by_groups(rules, 10_000, 100, 1_000, *E5M3_64, k=128) and not _by_groups(rules, 10_000, 100, 1_000, *E5M3_64, k=129)
    assert _by_groups(rules, 16_384, 100, 1_000, *E5M3_64) and not _by_groups(rules, 16_385, 100, 1_000, *E5M3_64)
    assert not _by_groups(rules, 10_000, 100, 1_000, 8, 64, 4, 0, False)
    assert not rules.by_groups(10_000, 10, 0, 0.0, 0.0, 0.0, 8, 64, 1, 4, True)          # an index without vectors
