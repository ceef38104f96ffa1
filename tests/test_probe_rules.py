"""CPU checks of the rules by which a search chooses among the kernels of its probe selection: the library's own header, compiled on the spot."""
import ctypes
import os
import subprocess

import pytest

SHIM = """
#include "ivfpq_probe_rules.hpp"
extern "C" int big_tiles(int nq, int n_lists) { return ivfpq::coarse_big_tiles(nq, n_lists); }
extern "C" int strip_width(int nq, int n_lists) { return ivfpq::coarse_strip_width(nq, n_lists); }
extern "C" int use_strips(int nq, int n_lists, int k) { return ivfpq::coarse_use_strips(nq, n_lists, k); }
extern "C" int by_waves(int nq, int n_probes, double crowd) { return ivfpq::select_by_waves(nq, n_probes, crowd); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    where = tmp_path_factory.mktemp("rules")
    (where / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_06672_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, str(where / "shim.cpp"), "-o", str(where / "shim.so")], check=True)
    lib = ctypes.CDLL(str(where / "shim.so"))
    lib.by_waves.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_double]
    return lib


def test_middling_batches_are_ranked_in_fp32(rules):
    # fewer than 1,024 tiles of 128 x 128: the operands' products in fp32, strips of 32
    for nq, n_lists in ((10_000, 1024), (8_065, 1024), (16_256, 1024), (10_000, 1_500), (4_096, 2_000), (2_000, 8_000)):
        assert 512 <= -(-nq // 128) * -(-n_lists // 128) < 1024
        assert not rules.big_tiles(nq, n_lists) and rules.strip_width(nq, n_lists) == 32
    for nq, n_lists in ((16_257, 1024), (10_000, 1_665), (10_000, 50_000)):
        assert rules.big_tiles(nq, n_lists) and rules.strip_width(nq, n_lists) == 64
    # ... so that 100 probes of 8,192 clusters read strip summaries there
    assert rules.use_strips(1_100, 8_192, 100) and not rules.use_strips(1_100, 8_192, 129) and not rules.use_strips(8_192, 8_192, 65)


def test_a_wave_per_query_where_the_chip_is_full(rules):
    # up to 1,536 queries every workgroup is resident, and one selects faster than a wave (513 queries, 64 probes, 960 components: 73 us to 99)
    assert not any(rules.by_waves(nq, p, 20) for nq in (513, 777, 1_200, 1_536) for p in (1, 10, 64))
    assert all(rules.by_waves(nq, p, 20) for nq in (1_537, 2_000, 10_000) for p in (1, 10, 64))
    assert not rules.by_waves(10_000, 65, 20)


def test_crowded_clusters_are_left_to_workgroups(rules):
    # hundreds of clusters within the error bound: a wave's rounds take up to 2.4 times a workgroup's selection (1,600 queries, 64 probes)
    assert rules.by_waves(1_600, 64, 110) and not rules.by_waves(1_600, 64, 160) and not rules.by_waves(3_000, 64, 250)
    assert rules.by_waves(10_000, 64, 180) and not rules.by_waves(10_000, 64, 400)
