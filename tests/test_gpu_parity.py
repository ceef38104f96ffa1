"""GPU parity: the HIP library against the CPU oracle, element by element, on the same seeded
inputs, through the C ABI (ctypes binding).  Every test here needs an MI355X.

Bars (stated here, used below):
  * table entries for half and e5m3: the stored bytes are identical to the oracle's;
    the fp32 table too (same fp32 operation order on both sides);
  * accumulated distances R: within 1e-5 relative (fp32 adds of <= 64 non-negative terms in the
    same order; the tolerance leaves room for a different summation order);
  * top-k ids: equal except inside ties within that tolerance; padding identical;
  * probe lists: same clusters rank by rank, swaps only between clusters whose float64
    distances agree to 1e-5 relative.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from util_parity import (RTOL, assert_probes_match, assert_topk_matches, oracle_tiny_index, random_pair,
                         to_library)

pytestmark = pytest.mark.gpu

DTYPES = [oracle.LUT_FP32, oracle.LUT_FP16, oracle.LUT_E5M3]


@pytest.fixture(scope="module")
def P():
    import paper_2301_06672_amd as pkg
    pkg.lib()
    assert torch.cuda.is_available()
    return pkg


@pytest.fixture(scope="module")
def tiny(P):
    w, data, oidx = oracle_tiny_index()
    return w, data, oidx, to_library(P, oidx)


@pytest.fixture(params=[0, 2, 3], ids=["own-route", "in-order", "grouped"])
def route(P, request, monkeypatch):
    """Runs a test on the library's own route (at these sizes: all probes in one unfiltered launch), and with every
    index it uploads sent through the filtered scan in query order and grouped by cluster, which batches take."""
    upload = P.Index.ivfpq_upload

    def routed(self, *args, **kw):
        upload(self, *args, **kw)
        self.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, request.param)
        return self
    monkeypatch.setattr(P.Index, "ivfpq_upload", routed)
    shared = [request.getfixturevalue("tiny")[3]] if "tiny" in request.fixturenames else []
    for gidx in shared:
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, request.param)
    yield request.param
    for gidx in shared:
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, 0)


def _step(msg):
    print(f"[parity] {msg}", flush=True)


# ---------------------------------------------------------------- table entries (search steps 2-3)

@pytest.mark.parametrize("dtype", DTYPES)
def test_lut_bytes_identical_tiny(P, tiny, dtype):
    w, data, oidx, gidx = tiny
    q = si.queries(w, 16)
    for qi in range(0, 16, 3):
        for l in (0, 7, 63):
            _step(f"dump_lut dtype={dtype} q={qi} list={l}")
            got = gidx.ivfpq_dump_lut(q[qi], l, dtype).cpu().numpy()
            want, _ = oracle.lut_store(oracle.lut_f32(oidx, q[qi], l), dtype)
            np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("d,pq_dim,pq_bits", [(32, 32, 8), (32, 16, 8), (32, 8, 8), (48, 16, 8), (24, 8, 4),
                                              (128, 64, 8), (96, 48, 8), (128, 64, 4), (128, 32, 8),
                                              (64, 32, 5), (96, 16, 6), (128, 64, 6), (64, 32, 7), (128, 64, 7)])
def test_lut_bytes_identical_shapes_and_ranges(P, d, pq_dim, pq_bits):
    # sub-vector lengths 1, 2, 4 (templated) and 3 (generic); value scales that reach below the
    # smallest e5m3 value, into the half subnormals, and above the largest half / e5m3 value
    for scale in (1e-3, 1.0, 300.0):
        oidx, gidx = random_pair(P, 300, d, 3, pq_dim, pq_bits, salt=100 + d + pq_dim, scale=scale)
        q = (scale * np.random.default_rng(d).standard_normal(d)).astype(np.float32)
        for dtype in DTYPES:
            _step(f"dump_lut d={d} s={pq_dim} p={pq_bits} scale={scale} dtype={dtype}")
            got = gidx.ivfpq_dump_lut(q, 1, dtype).cpu().numpy()
            F = oracle.lut_f32(oidx, q, 1)
            want, _ = oracle.lut_store(F, dtype)
            np.testing.assert_array_equal(got, want)
        if scale == 300.0:
            assert F.max() > 122880.0      # the saturating end was exercised
        if scale == 1e-3:
            assert F.min() < 2.0 ** -15     # and the flooring end


@pytest.mark.usefixtures("route")
@pytest.mark.parametrize("bias", [-2, 1, 7, 14])
def test_e4m4_lut_bytes_and_search(P, tiny, bias):
    # the 4+4 split with a caller-chosen exponent bias: table bytes identical, search results as the oracle's
    w, data, oidx, gidx = tiny
    gidx.ivfpq_set_e4m4_bias(bias)
    q = si.queries(w, 40)
    for l in (3, 40):
        _step(f"e4m4 bias={bias} dump_lut list={l}")
        got = gidx.ivfpq_dump_lut(q[2], l, P.LUT_FP8_E4M4).cpu().numpy()
        want, _ = oracle.lut_store(oracle.lut_f32(oidx, q[2], l), oracle.LUT_E4M4, e4m4_bias=bias)
        np.testing.assert_array_equal(got, want)
    ids_g, d_g = gidx.ivfpq_search(q, w.n_probes, w.k, P.LUT_FP8_E4M4)
    probes, _ = gidx.ivfpq_select_probes(q, w.n_probes)
    ids_o, d_o = oracle.search(oidx, q, w.n_probes, w.k, oracle.LUT_E4M4, probes=probes.cpu().numpy().view(np.uint32),
                               e4m4_bias=bias)
    assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context=f"e4m4 bias={bias}")
    gidx.ivfpq_set_e4m4_bias(7)


@pytest.mark.usefixtures("route")
def test_e4m4_other_shapes(P):
    for d, pq_dim, pq_bits in ((128, 64, 4), (128, 32, 8), (24, 8, 4)):
        oidx, gidx = random_pair(P, 2000, d, 5, pq_dim, pq_bits, salt=900 + d + pq_bits)
        gidx.ivfpq_set_e4m4_bias(5)
        q = np.random.default_rng(900).standard_normal((20, d)).astype(np.float32)
        _step(f"e4m4 d={d} s={pq_dim} p={pq_bits}")
        ids_g, d_g = gidx.ivfpq_search(q, 3, 20, P.LUT_FP8_E4M4)
        probes, _ = gidx.ivfpq_select_probes(q, 3)
        ids_o, d_o = oracle.search(oidx, q, 3, 20, oracle.LUT_E4M4, probes=probes.cpu().numpy().view(np.uint32), e4m4_bias=5)
        assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context=f"e4m4 d={d} p={pq_bits}")


FP8 = {oracle.LUT_E5M3: "e5m3", oracle.LUT_E4M4: "e4m4"}


def _reset_fp8(P, gidx):
    gidx.ivfpq_set_fp8_encoding(P.LUT_FP8_E5M3, 15)
    gidx.ivfpq_set_fp8_encoding(P.LUT_FP8_E4M4, 7)


@pytest.mark.usefixtures("route")
@pytest.mark.parametrize("dtype", list(FP8))
@pytest.mark.parametrize("bias,trunc,per_table", [(15, True, False), (22, False, False), (3, True, False),
                                                  (0, False, True), (0, True, True)])
def test_fp8_encoding_options_lut_bytes_and_search(P, tiny, dtype, bias, trunc, per_table):
    # general exponent bias, truncating encode and per-table bias of both 8-bit formats: the table
    # bytes are identical to the oracle's and the search returns what the oracle returns
    w, data, oidx, gidx = tiny
    gidx.ivfpq_set_fp8_encoding(dtype, bias, P.ROUND_TRUNCATE if trunc else P.ROUND_NEAREST, per_table)
    try:
        q = si.queries(w, 40)
        kw = dict(truncate=trunc, bias=bias, per_table=per_table)
        for qi, l in ((2, 3), (5, 40), (11, 63)):
            _step(f"{FP8[dtype]} {kw} dump_lut q={qi} list={l}")
            got = gidx.ivfpq_dump_lut(q[qi], l, dtype).cpu().numpy()
            want, _ = oracle.lut_store(oracle.lut_f32(oidx, q[qi], l), dtype, **kw)
            np.testing.assert_array_equal(got, want)
        _step(f"{FP8[dtype]} {kw} search")
        ids_g, d_g = gidx.ivfpq_search(q, w.n_probes, w.k, dtype)
        probes, _ = gidx.ivfpq_select_probes(q, w.n_probes)
        ids_o, d_o = oracle.search(oidx, q, w.n_probes, w.k, dtype, probes=probes.cpu().numpy().view(np.uint32), **kw)
        assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context=f"{FP8[dtype]} {kw}")
    finally:
        _reset_fp8(P, gidx)


@pytest.mark.parametrize("d,pq_dim,pq_bits", [(32, 32, 8), (48, 16, 8), (24, 8, 4), (128, 64, 4), (96, 48, 8)])
def test_per_table_bias_shapes_and_ranges(P, d, pq_dim, pq_bits):
    # every table-building code path (sub-vector lengths 1, 2, 3, 4; 4- and 8-bit codes) at value scales
    # from far below to far above the fixed formats' ranges; with a per-table bias the bytes follow the scale
    ref = {}
    for scale in (2.0 ** -30, 1.0, 2.0 ** 20):
        oidx = oracle.make_index(d, 3, pq_dim, pq_bits, *si.random_index_arrays(300, d, 3, pq_dim, pq_bits, salt=100 + d + pq_dim))
        s = np.float32(scale)
        oidx_s = oracle.make_index(d, 3, pq_dim, pq_bits, oidx.centroids * s, oidx.codebooks * s, oidx.list_offsets,
                                   oidx.codes, oidx.ids)
        gidx = to_library(P, oidx_s)
        q = (np.random.default_rng(d).standard_normal(d)).astype(np.float32) * s
        F = oracle.lut_f32(oidx_s, q, 1)
        for dtype in FP8:
            for trunc in (False, True):
                gidx.ivfpq_set_fp8_encoding(dtype, 0, int(trunc), True)
                _step(f"per-table d={d} s={pq_dim} p={pq_bits} scale={scale} {FP8[dtype]} trunc={trunc}")
                got = gidx.ivfpq_dump_lut(q, 1, dtype).cpu().numpy()
                want, _ = oracle.lut_store(F, dtype, truncate=trunc, per_table=True)
                np.testing.assert_array_equal(got, want)
                key = (dtype, trunc)
                if key in ref:
                    np.testing.assert_array_equal(got, ref[key])     # scale invariance, on the GPU side too
                ref[key] = got
                R_g = gidx.ivfpq_scan_list(q, 1, dtype, int(oidx.list_offsets[2] - oidx.list_offsets[1])).cpu().numpy()
                _, dec = oracle.lut_store(F, dtype, truncate=trunc, per_table=True)
                R_o, _ = oracle.scan_list(oidx_s, dec, 1)
                np.testing.assert_allclose(R_g, R_o, rtol=RTOL, atol=0)


# ---------------------------------------------------------------- Eq. (1) over one cluster (step 4)

@pytest.mark.parametrize("dtype", DTYPES)
def test_scan_list_R_tiny(P, tiny, dtype):
    w, data, oidx, gidx = tiny
    q = si.queries(w, 4)
    sizes = np.diff(oidx.list_offsets)
    for l in (int(np.argmax(sizes)), int(np.argmin(sizes)), 5):
        _step(f"scan_list dtype={dtype} list={l} len={sizes[l]}")
        _, dec = oracle.lut_store(oracle.lut_f32(oidx, q[1], l), dtype)
        want, _ = oracle.scan_list(oidx, dec, l)
        got = gidx.ivfpq_scan_list(q[1], l, dtype, int(sizes[l])).cpu().numpy()
        np.testing.assert_allclose(got, want, rtol=RTOL, atol=0)


@pytest.mark.parametrize("d,pq_dim,pq_bits", [(128, 64, 8), (96, 48, 8), (128, 64, 4), (128, 32, 8), (32, 16, 8),
                                              (24, 24, 8), (24, 8, 4), (160, 80, 8),
                                              (64, 32, 5), (96, 16, 6), (128, 64, 6), (64, 32, 7), (128, 64, 7), (256, 128, 5)])
def test_scan_list_R_code_widths(P, d, pq_dim, pq_bits):
    # 64/48/32/16-byte codes (16-byte chunk kernels) and 24/4/80-byte codes (generic 4-byte path);
    # bit-packed 5/6/7-bit codes whose fields straddle words (20/12/28/56/80 bytes on the 4-byte path,
    # 48 bytes of 6-bit codes on the 16-byte path);
    # list lengths that span several 64-vector groups with a ragged tail
    oidx, gidx = random_pair(P, 1500, d, 4, pq_dim, pq_bits, salt=200 + d + pq_bits)
    q = np.random.default_rng(pq_dim).standard_normal(d).astype(np.float32)
    sizes = np.diff(oidx.list_offsets)
    for dtype in DTYPES:
        for l in range(4):
            _step(f"scan_list d={d} s={pq_dim} p={pq_bits} dtype={dtype} list={l} len={sizes[l]}")
            _, dec = oracle.lut_store(oracle.lut_f32(oidx, q, l), dtype)
            want, _ = oracle.scan_list(oidx, dec, l)
            got = gidx.ivfpq_scan_list(q, l, dtype, int(sizes[l])).cpu().numpy()
            np.testing.assert_allclose(got, want, rtol=RTOL, atol=0)


@pytest.mark.parametrize("n,d,pq_dim,pq_bits", [(1, 32, 16, 8), (63, 128, 64, 8), (65, 64, 32, 5), (700, 128, 64, 8),
                                                (2311, 128, 64, 8), (2311, 128, 64, 6), (1500, 24, 24, 8)])
def test_upload_places_every_code(P, n, d, pq_dim, pq_bits):
    # the codes travel n * 8 / code_bytes vectors at a time (64 at least): one trip, and several that end inside lists
    # and between them; empty lists at both ends and in a row in the middle
    n_lists = 24
    arrays = si.random_index_arrays(n, d, n_lists, pq_dim, pq_bits, salt=n, empty_lists=(0, 1, 9, 10, 11, 23))
    oidx = oracle.make_index(d, n_lists, pq_dim, pq_bits, *arrays)
    gidx = P.Index.ivfpq_index_from_arrays(d, n_lists, pq_dim, pq_bits, *arrays).ivfpq_upload()
    q = np.random.default_rng(n).standard_normal(d).astype(np.float32)
    for l in range(n_lists):
        size = int(oidx.list_offsets[l + 1] - oidx.list_offsets[l])
        _step(f"uploaded n={n} s={pq_dim} p={pq_bits} list={l} len={size}")
        want, _ = oracle.scan_list(oidx, oracle.lut_f32(oidx, q, l), l)
        np.testing.assert_allclose(gidx.ivfpq_scan_list(q, l, P.LUT_FP32, size).cpu().numpy(), want, rtol=RTOL, atol=0)


# ---------------------------------------------------------------- probe selection (step 1)

@pytest.mark.parametrize("n_probes", [1, 8, 64])
def test_select_probes_tiny(P, tiny, n_probes):
    w, data, oidx, gidx = tiny
    q = si.queries(w, 300)
    _step(f"select_probes P={n_probes}")
    probes, pd = gidx.ivfpq_select_probes(q, n_probes)
    probes = probes.cpu().numpy().view(np.uint32)
    assert_probes_match(probes, oidx.centroids, q, n_probes)
    want, want_d = oracle.select_probes(oidx, q, n_probes)
    np.testing.assert_allclose(pd.cpu().numpy(), want_d, rtol=RTOL)
    assert (probes == want).mean() > 0.999


def test_select_probes_many_lists_and_exact_ties(P):
    # 3000 clusters (does not fit one pass of anything), 96 dims, duplicated centroids -> exact ties
    arrays = list(si.random_index_arrays(64, 96, 3000, 48, 8, salt=300))
    arrays[0][100:110] = arrays[0][50]          # ten copies of centroid 50
    oidx = oracle.make_index(96, 3000, 48, 8, *arrays)
    gidx = to_library(P, oidx)
    rng = np.random.default_rng(300)
    q = rng.standard_normal((40, 96)).astype(np.float32)
    q[:5] = arrays[0][50] + 0.01 * rng.standard_normal((5, 96)).astype(np.float32)
    for n_probes in (5, 200, 1000):
        _step(f"select_probes L=3000 P={n_probes}")
        probes, _ = gidx.ivfpq_select_probes(q, n_probes)
        probes = probes.cpu().numpy().view(np.uint32)
        assert_probes_match(probes, oidx.centroids, q, n_probes)
    # the tie group must come out in ascending cluster index
    probes, _ = gidx.ivfpq_select_probes(q[:5], 11)
    for row in probes.cpu().numpy().view(np.uint32):
        np.testing.assert_array_equal(row, [50] + list(range(100, 110)))


def test_select_probes_6000_lists_ties_and_outliers(P):
    # 6000 clusters: the bound of the n_probes-th ranking value comes from a sample of the row that grows
    # with n_probes.  Duplicated centroids far apart in the row give exact ties; a query far from
    # everything and one on a centroid are included.
    arrays = list(si.random_index_arrays(7000, 64, 6000, 32, 8, salt=310))
    arrays[0][5000:5006] = arrays[0][40]        # copies of a sampled centroid among the unsampled ones
    arrays[0][3000] = arrays[0][2999]
    oidx = oracle.make_index(64, 6000, 32, 8, *arrays)
    gidx = to_library(P, oidx)
    rng = np.random.default_rng(310)
    q = rng.standard_normal((70, 64)).astype(np.float32)
    q[:4] = arrays[0][40] + 0.01 * rng.standard_normal((4, 64)).astype(np.float32)
    q[4] = arrays[0][5500]
    q[5] = 50.0
    for n_probes in (1, 7, 64, 300, 1000):
        _step(f"select_probes L=6000 P={n_probes}")
        probes, pd = gidx.ivfpq_select_probes(q, n_probes)
        probes = probes.cpu().numpy().view(np.uint32)
        assert_probes_match(probes, oidx.centroids, q, n_probes)
        want, want_d = oracle.select_probes(oidx, q, n_probes)
        np.testing.assert_allclose(pd.cpu().numpy(), want_d, rtol=RTOL)
    probes, _ = gidx.ivfpq_select_probes(q[:4], 7)
    for row in probes.cpu().numpy().view(np.uint32):
        np.testing.assert_array_equal(row, [40] + list(range(5000, 5006)))
    for dtype in (oracle.LUT_FP32, oracle.LUT_E5M3):
        ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, 64, 20, dtype)
        assert_topk_matches(ids_g, d_g, ids_o, d_o, context=f"6000 lists dtype={dtype}")


@pytest.mark.parametrize("n_lists,d,pq_dim", [(1, 20, 4), (33, 20, 4), (1024, 128, 64), (1025, 300, 4), (8192, 96, 48)])
def test_select_probes_direct_and_ranked_agree(P, n_lists, d, pq_dim):
    # few queries get every cluster's distance, more of them ranking values and a short list: the same lists and the same
    # bits, at odd numbers of components (one and several pieces of the queries) and on both sides of the rule's lines
    arrays = list(si.random_index_arrays(64, d, n_lists, pq_dim, 8, salt=330 + n_lists))
    if n_lists > 40:
        arrays[0][31:33] = arrays[0][5]
    gidx = to_library(P, oracle.make_index(d, n_lists, pq_dim, 8, *arrays))
    rng = np.random.default_rng(330)
    q = rng.standard_normal((513, d)).astype(np.float32)
    q[:3] = arrays[0][min(5, n_lists - 1)] + 0.01 * rng.standard_normal((3, d)).astype(np.float32)
    q[3, 1] = np.inf
    q[4, d - 1] = np.nan
    for n_probes in sorted({1, min(n_lists, 20), min(n_lists, 1000)}):
        _step(f"select_probes L={n_lists} d={d} P={n_probes}")
        probes, pd = (x.cpu().numpy() for x in gidx.ivfpq_select_probes(q, n_probes))
        exact = ((q[:64, None].astype(np.float64) - arrays[0][probes[:64]]) ** 2).sum(-1)
        np.testing.assert_allclose(pd[:64], exact, rtol=RTOL)
        for nq in (1, 2, 9, 24, 512):
            few, few_d = (x.cpu().numpy() for x in gidx.ivfpq_select_probes(q[:nq], n_probes))
            np.testing.assert_array_equal(few, probes[:nq])
            np.testing.assert_array_equal(few_d.view(np.uint32), pd[:nq].view(np.uint32))


def test_select_probes_strip_minima_large_batch(P):
    # enough queries x clusters that the ranking GEMM runs its 128 x 128 tiles and hands the selection
    # the minima of 64-cluster strips; n_probes on both sides of the rule that decides whether they are used
    arrays = list(si.random_index_arrays(7000, 32, 6000, 16, 8, salt=320))
    arrays[0][5990:5996] = arrays[0][17]        # exact ties across strips, one in the ragged last strip
    oidx = oracle.make_index(32, 6000, 16, 8, *arrays)
    gidx = to_library(P, oidx)
    rng = np.random.default_rng(320)
    q = rng.standard_normal((3000, 32)).astype(np.float32)
    q[:6] = arrays[0][17] + 0.01 * rng.standard_normal((6, 32)).astype(np.float32)
    for n_probes in (1, 7, 47, 48, 200):
        _step(f"select_probes strips L=6000 nq=3000 P={n_probes}")
        probes, pd = gidx.ivfpq_select_probes(q, n_probes)
        probes = probes.cpu().numpy().view(np.uint32)
        want, want_d = oracle.select_probes(oidx, q, n_probes)
        np.testing.assert_allclose(pd.cpu().numpy(), want_d, rtol=RTOL)
        assert (probes == want).mean() > 0.999
        assert all(len(set(r)) == n_probes for r in probes[:200])
    probes, _ = gidx.ivfpq_select_probes(q, 7)
    for row in probes.cpu().numpy().view(np.uint32)[:6]:
        np.testing.assert_array_equal(row, [17] + list(range(5990, 5996)))


def test_select_probes_bf16_tiles_with_padded_dimension(P):
    # d = 24 is not a multiple of the 16-component slices of the bf16 kernel: the split pads with zeros
    arrays = list(si.random_index_arrays(7000, 24, 6000, 12, 8, salt=340))
    oidx = oracle.make_index(24, 6000, 12, 8, *arrays)
    gidx = to_library(P, oidx)
    q = np.random.default_rng(340).standard_normal((3000, 24)).astype(np.float32)
    for n_probes in (5, 33):
        _step(f"select_probes d=24 L=6000 nq=3000 P={n_probes}")
        probes, pd = gidx.ivfpq_select_probes(q, n_probes)
        want, want_d = oracle.select_probes(oidx, q, n_probes)
        np.testing.assert_allclose(pd.cpu().numpy(), want_d, rtol=RTOL)
        assert (probes.cpu().numpy().view(np.uint32) == want).mean() > 0.999


@pytest.mark.usefixtures("route")
@pytest.mark.parametrize("nq", [40, 3000])
def test_non_finite_queries_stay_in_range(P, nq):
    # NaN, infinite and huge queries: the call returns, every index it returns is valid, and the finite
    # queries of the same batch get their exact answer (40 queries: fp32 tiles and all ranking keys;
    # 3000: bf16 tiles and strip summaries)
    arrays = list(si.random_index_arrays(7000, 32, 6000, 16, 8, salt=350))
    oidx = oracle.make_index(32, 6000, 16, 8, *arrays)
    gidx = to_library(P, oidx)
    q = np.random.default_rng(350).standard_normal((nq, 32)).astype(np.float32)
    bad = [1, 7, 20, 33]
    q[1, 3] = np.nan
    q[7, :] = np.inf
    q[20, 0] = -np.inf
    q[33, :] = 3.0e38
    good = np.setdiff1d(np.arange(nq), bad)
    _step(f"non-finite queries nq={nq}: probes")
    probes, _ = gidx.ivfpq_select_probes(q, 12)
    probes = probes.cpu().numpy().view(np.uint32)
    assert probes.max() < 6000
    want, _ = oracle.select_probes(oidx, q[good], 12)
    assert (probes[good] == want).mean() > 0.999
    _step(f"non-finite queries nq={nq}: search")
    ids, dist = gidx.ivfpq_search(q, 12, 10, P.LUT_FP8_E5M3)
    ids = ids.cpu().numpy()
    assert ids.min() >= -1 and ids.max() < 7000
    ids_o, d_o = oracle.search(oidx, q[good], 12, 10, oracle.LUT_E5M3, probes=probes[good])
    assert_topk_matches(ids[good], dist.cpu().numpy()[good], ids_o, d_o, context="finite queries beside non-finite ones")


def test_select_probes_plateau_of_equal_centroids(P):
    # 40,000 clusters, all but three with the same centroid: every strip minimum equals the bound, more
    # strips qualify than the list holds, the whole row overflows the candidate buffer and the kernel
    # ends in its exact whole-row selection; ties come out by ascending cluster index
    arrays = list(si.random_index_arrays(41000, 8, 40000, 4, 8, salt=330))
    arrays[0][:] = arrays[0][0]
    arrays[0][[12345, 777, 39999]] += np.float32(0.25)
    oidx = oracle.make_index(8, 40000, 4, 8, *arrays)
    gidx = to_library(P, oidx)
    q = np.tile(arrays[0][12345], (3, 1)).astype(np.float32)
    q[1] = arrays[0][0]
    for n_probes in (1, 10, 300):
        _step(f"select_probes plateau P={n_probes}")
        probes, pd = gidx.ivfpq_select_probes(q, n_probes)
        probes = probes.cpu().numpy().view(np.uint32)
        want, want_d = oracle.select_probes(oidx, q, n_probes)
        np.testing.assert_array_equal(probes, want)
        np.testing.assert_allclose(pd.cpu().numpy(), want_d, rtol=RTOL)


# ---------------------------------------------------------------- whole search (steps 1-5)

def _search_both(gidx, oidx, q, n_probes, k, dtype):
    """GPU search; the oracle is run on the GPU's probe lists so that a near-tie in step 1 does not
    turn into a different (and equally valid) candidate set downstream."""
    ids_g, d_g = gidx.ivfpq_search(q, n_probes, k, dtype)
    probes, _ = gidx.ivfpq_select_probes(q, n_probes)
    probes = probes.cpu().numpy().view(np.uint32)
    ids_o, d_o = oracle.search(oidx, q, n_probes, k, dtype, probes=probes)
    return ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o


@pytest.mark.usefixtures("route")
@pytest.mark.parametrize("dtype", DTYPES)
def test_search_tiny_config(P, tiny, dtype):
    w, data, oidx, gidx = tiny
    q = si.queries(w)                            # all 1,000 queries of the configuration
    _step(f"search tiny dtype={dtype}")
    ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, w.n_probes, w.k, dtype)
    swapped = assert_topk_matches(ids_g, d_g, ids_o, d_o, context=f"tiny dtype={dtype}")
    assert swapped <= 0.01 * ids_o.size
    # and against the oracle's own probe selection: same answer for (nearly) every query
    ids_oo, _ = oracle.search(oidx, q, w.n_probes, w.k, dtype)
    assert (ids_oo == ids_g).all(axis=1).mean() > 0.99
    gt, _ = oracle.exact_knn(data, q[:200], w.k)
    assert abs(oracle.recall(ids_g[:200], gt) - oracle.recall(ids_oo[:200], gt)) < 1e-3


@pytest.mark.usefixtures("route")
@pytest.mark.parametrize("n_probes,k", [(1, 1), (3, 100), (64, 10), (8, 1024)])
def test_search_tiny_probe_and_k_range(P, tiny, n_probes, k):
    w, data, oidx, gidx = tiny
    q = si.queries(w, 64)
    for dtype in (oracle.LUT_FP32, oracle.LUT_E5M3):
        _step(f"search tiny P={n_probes} k={k} dtype={dtype}")
        ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, n_probes, k, dtype)
        assert_topk_matches(ids_g, d_g, ids_o, d_o, context=f"P={n_probes} k={k} dtype={dtype}")


@pytest.mark.usefixtures("route")
@pytest.mark.parametrize("d,pq_dim,pq_bits", [(128, 64, 8), (96, 48, 8), (128, 64, 4), (128, 32, 8), (24, 8, 4),
                                              (64, 32, 5), (128, 64, 6), (32, 16, 6), (128, 64, 7)])
def test_search_random_index_ragged_and_empty_lists(P, d, pq_dim, pq_bits):
    oidx, gidx = random_pair(P, 5000, d, 37, pq_dim, pq_bits, salt=400 + d + pq_bits, empty_lists=(0, 5, 36))
    q = np.random.default_rng(400).standard_normal((50, d)).astype(np.float32)
    for dtype in DTYPES:
        for n_probes, k in ((4, 10), (37, 100)):
            _step(f"search random d={d} s={pq_dim} p={pq_bits} dtype={dtype} P={n_probes} k={k}")
            ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, n_probes, k, dtype)
            assert_topk_matches(ids_g, d_g, ids_o, d_o, context=f"d={d} p={pq_bits} dtype={dtype}")


@pytest.mark.usefixtures("route")
def test_search_fewer_candidates_than_k_pads(P):
    oidx, gidx = random_pair(P, 70, 32, 9, 16, 8, salt=500, empty_lists=(1, 2))
    q = np.random.default_rng(500).standard_normal((8, 32)).astype(np.float32)
    probes = np.tile(np.array([[1, 2, 3]], dtype=np.uint32), (8, 1))      # two empty clusters and a small one
    ids_g, d_g = gidx.ivfpq_search_with_probes(q, probes, 50, oracle.LUT_FP16)
    ids_o, d_o = oracle.search(oidx, q, 3, 50, oracle.LUT_FP16, probes=probes)
    assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context="padding")
    assert (ids_o == -1).any()
    probes = np.tile(np.array([[1, 2]], dtype=np.uint32), (8, 1))         # nothing to scan at all
    ids_g, d_g = gidx.ivfpq_search_with_probes(q, probes, 5, oracle.LUT_FP32)
    assert (ids_g.cpu().numpy() == -1).all() and np.isinf(d_g.cpu().numpy()).all()


@pytest.mark.usefixtures("route")
def test_search_massive_ties_order_by_id(P):
    # 6000 identical codes in one cluster: every R is equal, the answer is the k smallest ids
    # (more ties than the selection's LDS record capacity -> the 64-bit tie-key path)
    cent, cb, offs, codes, ids = si.random_index_arrays(6400, 32, 2, 16, 8, salt=600)
    codes[:] = codes[0]
    oidx = oracle.make_index(32, 2, 16, 8, cent, cb, offs, codes, ids)
    gidx = to_library(P, oidx)
    q = np.random.default_rng(600).standard_normal((3, 32)).astype(np.float32)
    for k in (1, 10, 1000):
        for n_probes in (1, 2):
            _step(f"massive ties k={k} P={n_probes}")
            ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, n_probes, k, oracle.LUT_E5M3)
            np.testing.assert_array_equal(ids_g, ids_o)
            np.testing.assert_array_equal(d_g, d_o)


@pytest.mark.usefixtures("route")
def test_search_small_nearest_cluster_admits_everything(P):
    # the nearest probe holds fewer than k vectors, so its R values give no bound: every vector of
    # the large second cluster survives the filter of the filtered routes (each wave appends several staged batches)
    n, d = 3300, 32
    cent, cb, _, codes, ids = si.random_index_arrays(n, d, 3, 16, 8, salt=800)
    offs = np.array([0, 40, 3240, 3300], dtype=np.int64)
    oidx = oracle.make_index(d, 3, 16, 8, cent, cb, offs, codes, ids)
    gidx = to_library(P, oidx)
    q = np.random.default_rng(800).standard_normal((6, d)).astype(np.float32)
    for probes_row, k in (([0, 1], 100), ([0, 1, 2], 1000), ([2, 1], 64), ([1, 0], 10)):
        probes = np.tile(np.array([probes_row], dtype=np.uint32), (6, 1))
        for dtype in (oracle.LUT_FP32, oracle.LUT_E5M3):
            _step(f"small nearest cluster probes={probes_row} k={k} dtype={dtype}")
            ids_g, d_g = gidx.ivfpq_search_with_probes(q, probes, k, dtype)
            ids_o, d_o = oracle.search(oidx, q, len(probes_row), k, dtype, probes=probes)
            assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context=f"probes={probes_row} k={k}")


@pytest.mark.usefixtures("route")
def test_search_cluster_listed_twice_is_scanned_twice(P, tiny):
    w, data, oidx, gidx = tiny
    q = si.queries(w, 10)
    probes = np.tile(np.array([[4, 4, 9]], dtype=np.uint32), (10, 1))
    ids_g, d_g = gidx.ivfpq_search_with_probes(q, probes, 20, oracle.LUT_FP32)
    ids_o, d_o = oracle.search(oidx, q, 3, 20, oracle.LUT_FP32, probes=probes)
    assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context="dup cluster")


@pytest.mark.usefixtures("route")
def test_empty_inputs(P, tiny):
    w, data, oidx, gidx = tiny
    ids, d = gidx.ivfpq_search(np.zeros((0, w.d), np.float32), 4, 10, oracle.LUT_E5M3)
    assert ids.shape == (0, 10) and d.shape == (0, 10)
    # an index with no vectors at all
    cent, cb, offs, codes, ids0 = si.random_index_arrays(0, 32, 4, 16, 8, salt=700)
    oidx0 = oracle.make_index(32, 4, 16, 8, cent, cb, offs, codes, ids0)
    g0 = to_library(P, oidx0)
    q = np.ones((3, 32), np.float32)
    ids, d = g0.ivfpq_search(q, 2, 5, oracle.LUT_FP32)
    assert (ids.cpu().numpy() == -1).all() and np.isinf(d.cpu().numpy()).all()


def test_error_paths(P, tiny):
    w, data, oidx, gidx = tiny
    q = torch.from_numpy(si.queries(w, 4)).cuda()
    with pytest.raises(P.IvfpqError) as e:
        gidx.ivfpq_search(q, 0, 10, 0)
    assert e.value.status == P.EINVAL
    with pytest.raises(P.IvfpqError) as e:
        gidx.ivfpq_search(q, w.n_lists + 1, 10, 0)
    assert e.value.status == P.EINVAL
    with pytest.raises(P.IvfpqError) as e:
        gidx.ivfpq_search(q, 4, P.MAX_K + 1, 0)
    assert e.value.status == P.EINVAL
    with pytest.raises(P.IvfpqError) as e:
        gidx.ivfpq_search(q, 4, 10, 7)
    assert e.value.status == P.EINVAL
    with pytest.raises(P.IvfpqError) as e:
        gidx.ivfpq_set_e4m4_bias(500)
    assert e.value.status == P.EINVAL
    for bad in ((P.LUT_FP16, 15, 0, 0), (P.LUT_FP8_E5M3, -97, 0, 0), (P.LUT_FP8_E5M3, 111, 0, 0),
                (P.LUT_FP8_E4M4, 7, 2, 0), (P.LUT_FP8_E4M4, 7, 0, 3)):
        with pytest.raises(P.IvfpqError) as e:
            gidx.ivfpq_set_fp8_encoding(*bad)
        assert e.value.status == P.EINVAL
    # a workspace that is too small is refused before anything is launched
    import ctypes
    ids = torch.empty((4, 10), dtype=torch.int64, device="cuda")
    d = torch.empty((4, 10), dtype=torch.float32, device="cuda")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    st = P.lib().ivfpq_search(gidx._h, ctypes.c_void_p(q.data_ptr()), 4, 4, 10, 0, ctypes.c_void_p(ids.data_ptr()),
                              ctypes.c_void_p(d.data_ptr()), ctypes.c_void_p(ws.data_ptr()), 256, None)
    assert st == P.ENOSPACE
    # no device image yet
    fresh = P.Index.ivfpq_index_from_arrays(oidx.d, oidx.n_lists, oidx.pq_dim, oidx.pq_bits, oidx.centroids,
                                            oidx.codebooks, oidx.list_offsets, oidx.codes, oidx.ids)
    with pytest.raises(P.IvfpqError) as e:
        fresh.ivfpq_search(q, 4, 10, 0)
    assert e.value.status == P.ESTATE


def test_stage_timing_reports(P, tiny):
    w, data, oidx, gidx = tiny
    q = torch.from_numpy(si.queries(w, 256)).cuda()
    gidx.ivfpq_set_stage_timing(True)
    gidx.ivfpq_search(q, 8, 10, oracle.LUT_E5M3)
    torch.cuda.synchronize()
    ms = gidx.ivfpq_stage_times_ms()
    gidx.ivfpq_set_stage_timing(False)
    assert ms["total"] > 0 and ms["scan"] > 0
    assert ms["probe_select"] + ms["scan"] + ms["topk"] <= ms["total"] * 1.05 + 0.05
    # single launches inside the stages
    assert 0 < ms["rank_gemm"] <= ms["probe_select"] * 1.05 + 0.05
    assert ms["scan_nearest_kernel"] > 0 and ms["scan_filtered_kernel"] > 0
    assert ms["scan_nearest_kernel"] + ms["scan_filtered_kernel"] <= ms["scan"] * 1.05 + 0.05


@pytest.mark.parametrize("share,one_launch", [(0, True), (1, False)])
def test_stage_times_of_single_launches_are_parts_of_their_stage(P, tiny, share, one_launch):
    # all probes in one launch (this little work, no knob set) and the grouped scan: the two entries never count the
    # same time twice.  The spans are nested in the scan stage's, so their sum cannot exceed it but for the rounding
    # of an event's time (the events tick every 10 ns at the finest; 1 us is allowed)
    w, data, oidx, gidx = tiny
    q = torch.from_numpy(si.queries(w, 256)).cuda()
    gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, share)
    gidx.ivfpq_set_stage_timing(True)
    try:
        for n_probes in (1, 8):
            _step(f"stage times share={share} P={n_probes}")
            gidx.ivfpq_search(q, n_probes, 10, oracle.LUT_E5M3)
            torch.cuda.synchronize()
            ms = gidx.ivfpq_stage_times_ms()
            near, rest = ms["scan_nearest_kernel"], ms["scan_filtered_kernel"]
            assert near > 0 and (rest > 0) == (n_probes > 1)
            assert near + rest <= ms["scan"] + 1e-3
            if one_launch:
                np.testing.assert_allclose(rest, near * (n_probes - 1), rtol=1e-5)
    finally:
        gidx.ivfpq_set_stage_timing(False)
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, 0)


def test_early_exit_knob_leaves_the_route_alone(P, tiny):
    # 128 queries x 8 probes of 156 vectors: all probes in one launch (the scan entries divide its time by the pairs),
    # whatever the early exit is set to; and the three routes can be asked for by name
    w, data, oidx, gidx = tiny
    q = torch.from_numpy(si.queries(w, 128)).cuda()
    gidx.ivfpq_set_stage_timing(True)

    def one_launch():
        gidx.ivfpq_search(q, 8, 10, oracle.LUT_E5M3)
        torch.cuda.synchronize()
        ms = gidx.ivfpq_stage_times_ms()
        return abs(ms["scan_filtered_kernel"] / ms["scan_nearest_kernel"] - 7.0) < 1e-4
    try:
        for early in (0, 1, -1):
            _step(f"route with early exit {early}")
            gidx.ivfpq_set_tuning(P.TUNE_EARLY_EXIT, early)
            assert one_launch()
        for route in (1, 2, 3):
            _step(f"route {route}")
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
            assert one_launch() == (route == 1)
    finally:
        gidx.ivfpq_set_stage_timing(False)
        gidx.ivfpq_set_tuning(P.TUNE_EARLY_EXIT, 0)
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, 0)


def test_library_builder_index_searches_like_oracle_builder(P, tiny):
    # the two builders run different k-means code: compare them by recall only
    w, data, oidx, _ = tiny
    g = P.Index.ivfpq_build_host(data, w.n_lists, w.pq_dim, w.pq_bits, w.kmeans_iters, seed=3).ivfpq_upload()
    q = si.queries(w, 300)
    gt, _ = oracle.exact_knn(data, q, w.k)
    ids_lib, _ = g.ivfpq_search(q, w.n_probes, w.k, oracle.LUT_FP32)
    ids_orc, _ = oracle.search(oidx, q, w.n_probes, w.k, oracle.LUT_FP32)
    assert abs(oracle.recall(ids_lib.cpu().numpy(), gt) - oracle.recall(ids_orc, gt)) < 0.06


# ---------------------------------------------------------------- re-ranking with the stored vectors

def test_refine_matches_oracle(P, tiny):
    w, data, oidx, gidx = tiny
    q = si.queries(w, 200)
    x = torch.from_numpy(data).cuda()
    _step("refine: search k'=40, refine to 10")
    cand, _ = gidx.ivfpq_search(q, w.n_probes, 40, P.LUT_FP8_E5M3)
    ids_g, d_g = P.ivfpq_refine(x, q, cand, 10)
    ids_o, d_o = oracle.refine(data, q, cand.cpu().numpy(), 10)
    assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o.astype(np.float32), context="refine")
    gt, _ = oracle.exact_knn(data, q, 10)
    ids10, _ = gidx.ivfpq_search(q, w.n_probes, 10, P.LUT_FP8_E5M3)
    r0, r1 = oracle.recall(ids10.cpu().numpy(), gt), oracle.recall(ids_g.cpu().numpy(), gt)
    _step(f"refine: recall@10 {r0:.3f} -> {r1:.3f}")
    assert r1 > r0 + 0.03


@pytest.mark.parametrize("n_cand,k", [(1, 1), (7, 10), (64, 64), (1000, 100), (1024, 1024)])
def test_refine_edge_cases(P, n_cand, k):
    rng = np.random.default_rng(n_cand)
    n, d, nq = 3000, 24, 33
    data = rng.integers(-3, 4, size=(n, d)).astype(np.float32)      # integer grid: many exactly equal distances
    q = rng.integers(-3, 4, size=(nq, d)).astype(np.float32)
    cand = rng.integers(0, n, size=(nq, n_cand)).astype(np.int64)   # with duplicates
    cand[rng.random(cand.shape) < 0.2] = -1                          # padding entries anywhere
    if n_cand > 3:
        cand[5, :] = -1                                              # a query with no candidate at all
        cand[6, 3] = n + 5                                           # an id beyond the data: skipped
    _step(f"refine edge n_cand={n_cand} k={k}")
    ids_g, d_g = P.ivfpq_refine(torch.from_numpy(data).cuda(), q, torch.from_numpy(cand).cuda(), k)
    cand_o = np.where(cand >= n, -1, cand)
    ids_o, d_o = oracle.refine(data, q, cand_o, k)
    # integer-valued data: fp32 distances are exact, so the result is identical, ties by id included
    np.testing.assert_array_equal(ids_g.cpu().numpy(), ids_o)
    np.testing.assert_array_equal(d_g.cpu().numpy().astype(np.float64), d_o)


def test_refine_rejects_bad_arguments(P):
    x = torch.zeros((10, 8), device="cuda")
    q = torch.zeros((2, 8), device="cuda")
    for n_cand, k in ((P.MAX_K + 1, 5), (4, 0), (4, P.MAX_K + 1)):
        with pytest.raises(P.IvfpqError) as e:
            P.ivfpq_refine(x, q, torch.zeros((2, n_cand), dtype=torch.int64, device="cuda"), k)
        assert e.value.status == P.EINVAL


# ---------------------------------------------------------------- the streaming-read measurement kernel

@pytest.mark.parametrize("n_words,n_wg", [(4, 1), (4 * 1000, 3), (4 * 300001, 64)])
def test_stream_read_folds_every_word_once(P, n_words, n_wg):
    rng = np.random.default_rng(n_words)
    words = rng.integers(0, 2**32, size=n_words, dtype=np.uint64).astype(np.uint32)
    _step(f"stream read {n_words} words, {n_wg} workgroups")
    out = P.ivfpq_stream_read(torch.from_numpy(words.view(np.int32)).cuda(), n_wg).cpu().numpy().view(np.uint32)
    # 16-byte word i belongs to workgroup (i // 256) % n_wg
    w16 = np.bitwise_xor.reduce(words.reshape(-1, 4), axis=1)
    owner = (np.arange(w16.size) // 256) % n_wg
    want = np.zeros(n_wg, dtype=np.uint32)
    np.bitwise_xor.at(want, owner, w16)
    np.testing.assert_array_equal(out, want)


# ---------------------------------------------------------------- several pairs of one cluster per workgroup

@pytest.mark.parametrize("d,pq_dim,pq_bits,n_lists,n_probes,k", [
    (32, 16, 8, 7, 5, 10),        # m = 2, few clusters: most neighbouring pairs share theirs (runs of 4, 3, 2 and 1)
    (64, 16, 8, 33, 8, 100),      # m = 4
    (48, 48, 8, 200, 40, 10),     # m = 1, three 16-byte chunks, many seams between clusters
    (128, 64, 8, 3, 3, 1000),     # four chunks; two pairs per query: odd and even runs
    (128, 32, 8, 20, 12, 100),    # two chunks, m = 4: the shape of the 10^8-vector workload with 8-bit codes
    (128, 64, 4, 20, 12, 100),    # 4-bit codes, two chunks, m = 2: the shape of the 10^8-vector workload with 4-bit codes
    (32, 32, 4, 7, 5, 10),        # 4-bit codes, one chunk, m = 1
    (128, 32, 4, 33, 8, 1000),    # 4-bit codes, one chunk, m = 4
    (96, 96, 4, 50, 20, 10),      # 4-bit codes, three chunks
    (128, 128, 4, 9, 6, 100),     # 4-bit codes, four chunks
])
@pytest.mark.parametrize("dtype_name", ["e5m3", "e4m4", "fp16", "fp32"])
def test_search_group_of_pairs_per_workgroup(P, d, pq_dim, pq_bits, n_lists, n_probes, k, dtype_name):
    # the kernel that interleaves the tables of two or four queries of one cluster is forced on; results must be
    # those of the oracle, and identical to the one-pair kernel's (same arithmetic per query, same order)
    dtype = {"e5m3": oracle.LUT_E5M3, "e4m4": oracle.LUT_E4M4, "fp16": oracle.LUT_FP16, "fp32": oracle.LUT_FP32}[dtype_name]
    oidx, gidx = random_pair(P, 9000, d, n_lists, pq_dim, pq_bits, salt=900 + d, empty_lists=(1,) if n_lists > 3 else ())
    q = np.random.default_rng(900 + d).standard_normal((257, d)).astype(np.float32)
    gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, 1)
    assert gidx.ivfpq_scan_kernel_info(dtype).startswith("scan_kernel")
    ids_one, d_one = gidx.ivfpq_search(q, n_probes, k, dtype)
    for share in (2, 4):
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, share)
        info = gidx.ivfpq_scan_kernel_info(dtype)
        _step(f"{share} pairs per workgroup d={d} s={pq_dim} p={pq_bits} L={n_lists} P={n_probes} k={k} {dtype_name}: {info}")
        if not info.startswith("scan_group_kernel"):
            continue                      # tables of that many queries do not fit the LDS
        ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, n_probes, k, dtype)
        assert_topk_matches(ids_g, d_g, ids_o, d_o, context=f"{share} pairs per workgroup")
        np.testing.assert_array_equal(d_g, d_one.cpu().numpy())
        np.testing.assert_array_equal(ids_g, ids_one.cpu().numpy())
    gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, 0)


@pytest.mark.parametrize("n,d,pq_dim,pq_bits,n_lists,n_probes,nq,k", [
    (9000, 128, 64, 8, 20, 12, 1, 10),       # one query, every value of every probe
    (9000, 96, 48, 8, 20, 12, 257, 100),     # the same for many queries
    (9000, 64, 32, 7, 10, 8, 512, 10),       # 3.7 M vectors looked up: filtered, pairs in query order
    (9000, 64, 32, 5, 10, 8, 444, 10),       # 3.2 M less a little: whole rows still
    (9000, 64, 32, 5, 10, 8, 513, 1000),     # one query more than the large selection workgroups take
    (9000, 32, 16, 8, 10, 8, 800, 10),       # 5.8 M: in query order
    (9000, 32, 16, 8, 10, 8, 1010, 10),      # 7.3 M: pairs grouped by cluster
    (40000, 64, 64, 4, 8, 5, 40, 100),       # 25,000 vectors a query: filtered, in query order
    (300, 24, 24, 8, 6, 5, 33, 400),         # k above the candidates
    (5000, 32, 16, 8, 9, 1, 50, 10),         # a single probe
])
@pytest.mark.parametrize("dtype", [oracle.LUT_E5M3, oracle.LUT_FP16, oracle.LUT_FP32])
def test_scan_routes_agree(P, n, d, pq_dim, pq_bits, n_lists, n_probes, nq, k, dtype):
    # whichever way the probes are scanned (all values of all probes; filtered in query order; filtered and grouped, one or
    # several pairs per workgroup) every distance is the same sum in the same order: equal results, bit for bit
    oidx, gidx = random_pair(P, n, d, n_lists, pq_dim, pq_bits, salt=640 + nq, empty_lists=(2,))
    q = np.random.default_rng(nq).standard_normal((nq, d)).astype(np.float32)
    probes = np.stack([np.random.default_rng(i).permutation(n_lists)[:n_probes] for i in range(nq)]).astype(np.uint32)
    probes[0, -1] = 0xFFFFFFFF               # out of range: skipped
    probes[-1, -1] = probes[-1, 0]           # the same cluster twice
    out = {}
    ways = (("own", P.TUNE_SCAN_ROUTE, 0), ("whole rows", P.TUNE_SCAN_ROUTE, 1), ("in order", P.TUNE_SCAN_ROUTE, 2),
            ("grouped", P.TUNE_SCAN_ROUTE, 3), ("one pair", P.TUNE_SCAN_SHARE, 1))
    for name, knob, value in ways:
        gidx.ivfpq_set_tuning(knob, value)
        _step(f"routes n={n} s={pq_dim} p={pq_bits} P={n_probes} nq={nq} k={k} dtype={dtype}: {name}")
        out[name] = [t.cpu().numpy() for t in (*gidx.ivfpq_search(q, n_probes, k, dtype),
                                               *gidx.ivfpq_search_with_probes(q, probes, k, dtype),
                                               *gidx.ivfpq_search_static(q, n_probes, k, dtype))]
        gidx.ivfpq_set_tuning(knob, 0)
    for name, _, _ in ways[1:]:
        for a, b in zip(out["own"], out[name]):
            np.testing.assert_array_equal(a, b, err_msg=name)
    ids_o, d_o = oracle.search(oidx, q[:40], n_probes, k, dtype)
    assert_topk_matches(out["own"][0][:40], out["own"][1][:40], ids_o, d_o, context="own route")


@pytest.mark.parametrize("pq_bits,pq_dim", [(8, 32), (5, 32), (4, 16)])     # chunks of 16 and of 4 bytes
@pytest.mark.parametrize("n_probes", [1, 2, 6])
def test_first_probe_without_vectors(P, pq_bits, pq_dim, n_probes):
    # a query whose first probe is out of range, or an empty cluster, has no bound and no nearest segment: the other probes'
    # vectors are all it returns, and no centroid is looked up for a number that names none
    oidx, gidx = random_pair(P, 3000, 64, 9, pq_dim, pq_bits, salt=31, empty_lists=(2, 4))
    nq, k = 130, 20
    q = np.random.default_rng(31).standard_normal((nq, 64)).astype(np.float32)
    probes = np.stack([np.random.default_rng(i).permutation(9)[:n_probes] for i in range(nq)]).astype(np.uint32)
    skipped = np.zeros(nq, bool)
    for i, bad in ((0, 0xFFFFFFFF), (1, 9), (2, 1 << 30), (64, 0x80000000)):
        probes[i, 0], skipped[i] = bad, True
    probes[3, 0], probes[4, 0] = 2, 4
    probes[5] = 0xFFFFFFFE                    # none in range
    skipped[5] = True
    want = {}
    for dtype in DTYPES:
        for route in (0, 1, 2, 3):
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
            _step(f"first probe without vectors: p={pq_bits} P={n_probes} dtype={dtype} route={route}")
            got = [t.cpu().numpy() for t in gidx.ivfpq_search_with_probes(q, probes, k, dtype)]
            if dtype not in want:
                want[dtype] = got
            for a, b in zip(got, want[dtype]):
                np.testing.assert_array_equal(a, b)
        ids, dist = want[dtype]
        ok = ~skipped
        ids_o, d_o = oracle.search(oidx, q[ok], n_probes, k, dtype, probes=probes[ok])
        assert_topk_matches(ids[ok], dist[ok], ids_o, d_o, context="probes in range")
        for i in np.flatnonzero(skipped):     # the same query without that probe
            rest = probes[i:i + 1, 1:] if probes[i, -1] < 9 else probes[i:i + 1, :0]
            if rest.shape[1] == 0:
                assert np.all(ids[i] == -1) and np.all(np.isinf(dist[i]))
                continue
            ids_o, d_o = oracle.search(oidx, q[i:i + 1], n_probes - 1, k, dtype, probes=rest)
            assert_topk_matches(ids[i:i + 1], dist[i:i + 1], ids_o, d_o, context=f"query {i}")


@pytest.mark.parametrize("scale", [1e-22, 3e-22, 1e-21, 3e-21, 3e-20])
def test_distances_in_the_subnormal_range(P, scale):
    # R of a few to a few thousand units of 2^-149: the bins of the nearest probe's bound are narrower than one unit
    arrays = si.random_index_arrays(4000, 64, 8, 32, 8, salt=78, scale=scale)
    oidx = oracle.make_index(64, 8, 32, 8, *arrays)
    gidx = to_library(P, oidx)
    q = (scale * np.random.default_rng(78).standard_normal((65, 64))).astype(np.float32)
    for dtype in (oracle.LUT_FP32, oracle.LUT_E5M3):
        ids_o, d_o = oracle.search(oidx, q, 8, 20, dtype)
        for route in (0, 1, 2, 3):
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
            _step(f"subnormal distances, scale={scale} dtype={dtype} route={route}")
            ids_g, d_g = [t.cpu().numpy() for t in gidx.ivfpq_search(q, 8, 20, dtype)]
            np.testing.assert_array_equal(d_g.view(np.uint32), d_o.view(np.uint32))
            np.testing.assert_array_equal(ids_g, ids_o)


@pytest.mark.parametrize("d,pq_dim,pq_bits", [
    (128, 64, 8), (128, 32, 8), (96, 48, 8), (64, 32, 8), (64, 16, 8),     # two and four components a sub-space
    (96, 24, 8),                                                           # 24-byte codes: 4-byte chunks
    (128, 64, 4), (96, 48, 4), (128, 32, 4),                               # nibbles, in chunks of 16 and of 4 bytes
    (128, 64, 7), (128, 64, 6), (64, 32, 6), (128, 64, 5),                 # fields that straddle words
])
@pytest.mark.parametrize("scale", [1.0, 40.0])
def test_matrix_core_filter(P, d, pq_dim, pq_bits, scale):
    # Grouped batches list the vectors that can have R <= bound from products in bf16 and add up only those.  Survivors, order of
    # the sums and so every bit are those of the table kernels in query order.  Clusters of 0 to 1,025 vectors (work items of
    # 512, rounds of 32), pairs per cluster from 1 to beyond 64 (blocks of 32 rows); queries near a cluster, between clusters,
    # far outside, one not a number and one without a finite distance; k beyond the nearest cluster (no bound).  scale 40: half
    # tables and e4m4 saturate.
    sizes = [700, 0, 1, 31, 32, 33, 63, 64, 65, 511, 512, 513, 1025, 400, 900, 2, 640]
    rng = np.random.default_rng(1000 + d + pq_dim + pq_bits)
    n, L, m = sum(sizes), len(sizes), d // pq_dim
    cent = (rng.standard_normal((L, d)) * 2 * scale).astype(np.float32)
    book = (rng.standard_normal((pq_dim, 1 << pq_bits, m)) * 0.6 * scale).astype(np.float32)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    codes = rng.integers(0, 256, (n, pq_dim * pq_bits // 8), dtype=np.uint8)
    ids = rng.permutation(n).astype(np.int64)
    oidx = oracle.make_index(d, L, pq_dim, pq_bits, cent, book, offs, codes, ids)
    gidx = to_library(P, oidx)
    q = (cent[rng.integers(0, L, 230)] + rng.standard_normal((230, d)) * scale).astype(np.float32)
    q[40:80] = ((cent[rng.integers(0, L, 40)] + cent[rng.integers(0, L, 40)]) / 2).astype(np.float32)
    q[80:90] *= 30
    q[90, 3], q[91, 5] = np.nan, 3e38
    for dtype in (oracle.LUT_FP32, oracle.LUT_FP16, oracle.LUT_E5M3, oracle.LUT_E4M4):
        for nq, n_probes, k in ((230, 9, 10), (230, L, 100), (5, 4, 10), (33, 5, 700)):
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, 3)
            info = gidx.ivfpq_scan_kernel_info(dtype)
            top = {oracle.LUT_FP32: np.inf, oracle.LUT_FP16: 65504.0, oracle.LUT_E5M3: 122880.0, oracle.LUT_E4M4: 496.0}[dtype]
            assert info.startswith("scan_filter_kernel") == (4 * (book.astype(np.float64) ** 2).sum(2).max() <= top)
            _step(f"filter d={d} s={pq_dim} p={pq_bits} scale={scale} dtype={dtype} nq={nq} P={n_probes} k={k}")
            ids_f, d_f = [t.cpu().numpy() for t in gidx.ivfpq_search(q[:nq], n_probes, k, dtype)]
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, 2)
            ids_t, d_t = [t.cpu().numpy() for t in gidx.ivfpq_search(q[:nq], n_probes, k, dtype)]
            np.testing.assert_array_equal(d_f.view(np.uint32), d_t.view(np.uint32))
            np.testing.assert_array_equal(ids_f, ids_t)
            if nq == 230:
                ids_o, d_o = oracle.search(oidx, q[:40], n_probes, k, dtype)
                assert_topk_matches(ids_f[:40], d_f[:40], ids_o, d_o, context=info)


@pytest.mark.parametrize("dtype,bias", [(oracle.LUT_E5M3, 15), (oracle.LUT_E5M3, 24), (oracle.LUT_E5M3, 2), (oracle.LUT_E5M3, -96),
                                        (oracle.LUT_E4M4, 7), (oracle.LUT_E4M4, 12), (oracle.LUT_E4M4, 0), (oracle.LUT_E4M4, -100)])
@pytest.mark.parametrize("truncate", [False, True])
def test_matrix_core_filter_other_encodings(P, dtype, bias, truncate):
    # the filter's limit and the candidates' entries follow the encoding: biases that clamp small entries from below (all of them:
    # every sum is the same), rounding and truncation; the table kernels' bits
    oidx, gidx = random_pair(P, 6000, 128, 12, 64, 8, salt=79, empty_lists=(4,))
    gidx.ivfpq_set_fp8_encoding(dtype, bias, P.ROUND_TRUNCATE if truncate else P.ROUND_NEAREST)
    q = np.random.default_rng(79).standard_normal((222, 128)).astype(np.float32)
    got = []
    for route in (2, 3):
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
        _step(f"encoding dtype={dtype} bias={bias} truncate={truncate} route={route}: {gidx.ivfpq_scan_kernel_info(dtype)}")
        got.append([t.cpu().numpy() for t in gidx.ivfpq_search(q, 8, 20, dtype)])
    assert gidx.ivfpq_scan_kernel_info(dtype).startswith("scan_filter_kernel")
    np.testing.assert_array_equal(got[0][1].view(np.uint32), got[1][1].view(np.uint32))
    np.testing.assert_array_equal(got[0][0], got[1][0])


def test_matrix_core_filter_leaves_other_calls_to_the_tables(P):
    # encoding by a bias per table, knobs of the table kernels, queries that are not 8-byte aligned and codebooks that are no
    # moderate numbers: the table kernels, with the same results
    oidx, gidx = random_pair(P, 4000, 64, 9, 32, 8, salt=77)
    gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, 3)
    name = lambda: gidx.ivfpq_scan_kernel_info(oracle.LUT_E5M3).split("<")[0]
    assert name() == "scan_filter_kernel"
    for knob, value, back in ((P.TUNE_SCAN_SHARE, 2, 0), (P.TUNE_EARLY_EXIT, -1, 0), (P.TUNE_ORDER_BLOCK, 32, 0), (P.TUNE_SCAN_THREADS, 256, 0)):
        gidx.ivfpq_set_tuning(knob, value)
        assert name() == "scan_group_kernel"
        gidx.ivfpq_set_tuning(knob, back)
    q = np.random.default_rng(77).standard_normal((301, 64)).astype(np.float32)
    want = [t.cpu().numpy() for t in gidx.ivfpq_search(q, 6, 10, oracle.LUT_E5M3)]
    flat = torch.empty(q.size + 1, dtype=torch.float32, device="cuda")
    flat[1:] = torch.from_numpy(q).cuda().reshape(-1)
    got = [t.cpu().numpy() for t in gidx.ivfpq_search(flat[1:].view(301, 64), 6, 10, oracle.LUT_E5M3)]
    for a, b in zip(want, got):
        np.testing.assert_array_equal(a, b)
    gidx.ivfpq_set_fp8_encoding(oracle.LUT_E5M3, 15, P.ROUND_NEAREST, True)
    assert name() != "scan_filter_kernel"
    arrays = list(si.random_index_arrays(4000, 64, 9, 32, 8, salt=77))
    arrays[1] = arrays[1].copy()
    arrays[1][3, 7, 0] = np.inf
    odd = P.Index.ivfpq_index_from_arrays(64, 9, 32, 8, *arrays).ivfpq_upload()
    odd.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, 3)
    assert not odd.ivfpq_scan_kernel_info(oracle.LUT_FP32).startswith("scan_filter_kernel")


def test_timed_search_names_the_kernel_it_launched(P):
    # the general description does not know the batch, the probes and k; a timed search does
    oidx, gidx = random_pair(P, 70000, 64, 700, 32, 8, salt=5)
    name = lambda dtype: gidx.ivfpq_scan_kernel_info(dtype).split("<")[0]
    rng = np.random.default_rng(5)
    e5m3, half = oracle.LUT_E5M3, oracle.LUT_FP16
    assert name(e5m3) == name(half) == "scan_filter_kernel"
    gidx.ivfpq_set_stage_timing(True)
    assert name(e5m3) == "scan_filter_kernel"                           # no search yet
    for nq, n_probes, k, dtype, kernel in (
            (3, 5, 10, e5m3, "scan_kernel"),                            # little work: all probes in one launch
            (10000, 4, 10, e5m3, "scan_kernel"),                        # 4 M vectors: in query order
            (170000, 2, 10, e5m3, "scan_filter_kernel"),
            (170000, 2, 100, e5m3, "scan_group_kernel")):               # k a whole list
        q = rng.standard_normal((nq, 64)).astype(np.float32)
        gidx.ivfpq_search(q, n_probes, k, dtype)
        torch.cuda.synchronize()
        _step(f"nq={nq} P={n_probes} k={k} dtype={dtype}: {gidx.ivfpq_scan_kernel_info(dtype)}")
        assert name(dtype) == kernel
        assert name(half if dtype == e5m3 else e5m3) == "scan_filter_kernel"          # another dtype: the general description
    gidx.ivfpq_set_stage_timing(False)
    assert name(half) == "scan_filter_kernel"


@pytest.mark.parametrize("overlap", [False, True])
@pytest.mark.parametrize("d,pq_dim,pq_bits", [(128, 32, 8), (96, 48, 8), (128, 64, 7), (128, 64, 4)])
def test_filter_is_left_to_the_tables_where_lists_overlap(P, d, pq_dim, pq_bits, overlap):
    # the same sizes and the same call: lists around centroids far apart hold few vectors that can be among the results, those around
    # nearly one point as many as the nearest list does.  One empty list, and lists of 1 vector to thousands, are sampled
    # too.  Either way, the results of the other kernels, bit for bit.
    arrays = list(si.random_index_arrays(30000, d, 60, pq_dim, pq_bits, salt=91, empty_lists=(7,)))
    if overlap:
        arrays[0] = (0.02 * arrays[0]).astype(np.float32)
    gidx = to_library(P, oracle.make_index(d, 60, pq_dim, pq_bits, *arrays))
    rng = np.random.default_rng(91)
    cent = arrays[0][rng.integers(0, 60, 8000)]
    q = (cent + 0.3 * rng.standard_normal(cent.shape)).astype(np.float32)
    gidx.ivfpq_set_stage_timing(True)
    out = {}
    for dtype in (oracle.LUT_E5M3, oracle.LUT_FP32):
        for route in (0, 2, 3):
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
            out[route] = [t.cpu().numpy() for t in gidx.ivfpq_search(q, 20, 250, dtype)]
            name = gidx.ivfpq_scan_kernel_info(dtype)
            _step(f"d={d} p={pq_bits} overlap={overlap} dtype={dtype} route={route}: {name}")
            assert name.startswith("scan_filter_kernel") == (route == 3 or (route == 0 and not overlap))
        for a, b, c in zip(*out.values()):
            np.testing.assert_array_equal(a, b)
            np.testing.assert_array_equal(a, c)


def test_filter_is_left_to_the_tables_where_lists_have_few_pairs(P):
    # a block of 64 pairs costs the filter the same however few there are: 4 pairs a list of 2,000 vectors take the tables, 100 the
    # filter, with either call's results equal on both
    arrays = si.random_index_arrays(1600000, 128, 800, 32, 8, salt=93)
    gidx = to_library(P, oracle.make_index(128, 800, 32, 8, *arrays))
    rng = np.random.default_rng(93)
    gidx.ivfpq_set_stage_timing(True)
    dtype = oracle.LUT_E5M3
    for nq, kernel in ((320, "scan_group_kernel"), (8000, "scan_filter_kernel")):
        cent = arrays[0][rng.integers(0, 800, nq)]
        q = (cent + 0.3 * rng.standard_normal(cent.shape)).astype(np.float32)
        out = []
        for route, order_block, expected in ((0, 0, kernel), (3, 0, "scan_filter_kernel"), (3, 64, "scan_group_kernel")):
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
            gidx.ivfpq_set_tuning(P.TUNE_ORDER_BLOCK, order_block)
            out.append([t.cpu().numpy() for t in gidx.ivfpq_search(q, 11, 20, dtype)])
            name = gidx.ivfpq_scan_kernel_info(dtype)
            _step(f"nq={nq} route={route} order_block={order_block}: {name}")
            assert name.startswith(expected)
        gidx.ivfpq_set_tuning(P.TUNE_ORDER_BLOCK, 0)
        for other in out[1:]:
            np.testing.assert_array_equal(out[0][0], other[0])
            np.testing.assert_array_equal(out[0][1].view(np.uint32), other[1].view(np.uint32))


@pytest.mark.parametrize("nq", [1, 31, 33, 500, 2047, 2049])
def test_candidates_of_few_queries_are_shared_by_workgroups(P, nq):
    # long candidate lists (k a third of a list) of few queries are summed by several workgroups each, of many by one: every
    # listed vector is summed once, the same bits as a scan of every vector in query order
    oidx, gidx = random_pair(P, 20000, 64, 20, 32, 8, salt=870, empty_lists=(1,))
    q = np.random.default_rng(870).standard_normal((nq, 64)).astype(np.float32)
    got = []
    for route in (2, 3):
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
        _step(f"candidates nq={nq} route={route}")
        got.append([t.cpu().numpy() for t in gidx.ivfpq_search(q, 15, 300, oracle.LUT_E5M3)])
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1].view(np.uint32), got[1][1].view(np.uint32))


@pytest.mark.parametrize("d,pq_dim,pq_bits,n_lists,n_probes,k", [
    (64, 64, 5, 7, 5, 10),            # m = 1, 40-byte codes, few clusters: most neighbouring pairs share theirs
    (128, 64, 6, 20, 12, 100),        # m = 2, 48-byte codes in 16-byte chunks
    (128, 64, 7, 33, 8, 10),          # m = 2, 56-byte codes
    (256, 64, 7, 3, 3, 1000),         # m = 4; two pairs per query: odd and even runs
    (128, 64, 7, 200, 40, 10),        # many seams between clusters
    (32, 32, 5, 20, 12, 100),         # 20-byte codes: one unit of 32 fields, no split scan
    (64, 32, 6, 33, 8, 10),
    (128, 32, 7, 7, 5, 1000),
    (96, 48, 6, 20, 12, 10),          # 36-byte codes: three steps
    (96, 96, 7, 20, 12, 10),          # 84-byte codes: the first pass ends inside a unit of 32 fields
    (192, 96, 6, 33, 8, 100),
    (96, 96, 5, 7, 5, 10),
])
@pytest.mark.parametrize("dtype", [oracle.LUT_E5M3, oracle.LUT_E4M4, oracle.LUT_FP16, oracle.LUT_FP32])
def test_group_kernel_bit_packed_codes(P, d, pq_dim, pq_bits, n_lists, n_probes, k, dtype):
    # 5- to 7-bit codes: one pair per workgroup, two and four, and the library's choice, with the early
    # exit (tables built by halves) and without it, add the same entries in the same order: equal bits.  (8-bit tables of
    # 96 sub-spaces: the group kernel rounds once for two entries, the one-pair kernel twice, and the sums no longer fit
    # 24 bits: at most 96 roundings of 2^-24 each, which the tolerance of 1e-5 covers)
    oidx, gidx = random_pair(P, 9000, d, n_lists, pq_dim, pq_bits, salt=960 + d + pq_bits, empty_lists=(1,) if n_lists > 3 else ())
    q = np.random.default_rng(960 + d).standard_normal((257, d)).astype(np.float32)
    gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, 1)
    ids_one, d_one = [t.cpu().numpy() for t in gidx.ivfpq_search(q, n_probes, k, dtype)]
    ids_o, d_o = oracle.search(oidx, q[:40], n_probes, k, dtype)
    assert_topk_matches(ids_one[:40], d_one[:40], ids_o, d_o, context="one pair per workgroup")
    grouped = 0
    for share in (0, 2, 4):
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, share)
        info = gidx.ivfpq_scan_kernel_info(dtype)
        grouped += info.startswith("scan_group_kernel")
        for early in (1, -1):
            gidx.ivfpq_set_tuning(P.TUNE_EARLY_EXIT, early)
            _step(f"bit-packed d={d} s={pq_dim} p={pq_bits} L={n_lists} P={n_probes} k={k} dtype={dtype} share={share} early={early}: {info}")
            ids_g, d_g = [t.cpu().numpy() for t in gidx.ivfpq_search(q, n_probes, k, dtype)]
            if pq_dim > 64 and dtype in FP8:
                assert_topk_matches(ids_g, d_g, ids_one, d_one, context=info)
            else:
                np.testing.assert_array_equal(d_g, d_one)
                np.testing.assert_array_equal(ids_g, ids_one)
    assert grouped > 0


def test_group_kernel_survivor_overflow_and_small_batches(P):
    # a bound that admits everything (nearest cluster smaller than k) makes every vector of the big cluster a
    # survivor: groups with more survivors than a wave stages are appended directly; also 1, 2 and 3 queries
    # (slots that are not full) and a workspace limit that cuts the batch into tiles
    n, d = 21000, 64
    cent, cb, _, codes, ids = si.random_index_arrays(n, d, 3, 32, 8, salt=811)
    offs = np.array([0, 40, 20040, 21000], dtype=np.int64)
    oidx = oracle.make_index(d, 3, 32, 8, cent, cb, offs, codes, ids)
    gidx = to_library(P, oidx)
    rng = np.random.default_rng(811)
    for nq in (1, 2, 3, 9):
        q = (cent[0] + 0.01 * rng.standard_normal((nq, d))).astype(np.float32)       # nearest cluster: the 40-vector one
        for share in (2, 4):
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, share)
            for dtype in (oracle.LUT_E5M3, oracle.LUT_FP16):
                _step(f"overflow nq={nq} share={share} dtype={dtype}")
                ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, 3, 1000, dtype)
                assert_topk_matches(ids_g, d_g, ids_o, d_o, context="group kernel, every vector survives")
    gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, 0)


@pytest.mark.parametrize("d,pq_dim,pq_bits,dtype", [
    (128, 64, 8, oracle.LUT_E5M3), (128, 64, 8, oracle.LUT_FP32),     # four 16-byte chunks
    (96, 48, 8, oracle.LUT_FP16),                                     # three
    (64, 64, 4, oracle.LUT_E5M3),                                     # 4-bit codes: 32 sub-spaces per chunk
    (64, 32, 6, oracle.LUT_E4M4),                                     # 6-bit codes in 4-byte chunks
    (128, 64, 6, oracle.LUT_E5M3),                                    # 6-bit codes, 48 bytes: 16-byte chunks
    (40, 40, 8, oracle.LUT_E5M3),                                     # 40-byte codes: 4-byte chunks
])
def test_early_exit_changes_nothing(P, d, pq_dim, pq_bits, dtype):
    # a group whose partial sums are all over the bound stops early: the survivors, hence the results, are the same
    oidx, gidx = random_pair(P, 12000, d, 9, pq_dim, pq_bits, salt=950 + d + pq_bits)
    q = np.random.default_rng(950 + d).standard_normal((130, d)).astype(np.float32)
    for route in (2, 3):                 # the filtered routes: only they can stop early
        out = {}
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
        for mode in ("0", "1"):
            gidx.ivfpq_set_tuning(P.TUNE_EARLY_EXIT, 1 if mode == "1" else -1)
            _step(f"early exit {mode}: route={route} d={d} s={pq_dim} p={pq_bits} dtype={dtype}")
            ids, dist = gidx.ivfpq_search(q, 6, 10, dtype)
            out[mode] = (ids.cpu().numpy(), dist.cpu().numpy())
        np.testing.assert_array_equal(out["0"][0], out["1"][0])
        np.testing.assert_array_equal(out["0"][1], out["1"][1])
        gidx.ivfpq_set_tuning(P.TUNE_EARLY_EXIT, 0)
        ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, 6, 10, dtype)
        assert_topk_matches(ids_g, d_g, ids_o, d_o, context="early exit")


def test_split_scan_when_every_group_stays_in_the_race(P):
    # 64 sub-spaces of 8-bit codes: the filtered scan builds half the table first.  Here the nearest cluster
    # holds fewer than k vectors, so the bound admits everything: every group of the big cluster needs the
    # second half, more groups per wave than the first pass can note (it then takes them all again)
    n, d = 21000, 128
    cent, cb, _, codes, ids = si.random_index_arrays(n, d, 3, 64, 8, salt=810)
    offs = np.array([0, 40, 20040, 21000], dtype=np.int64)
    oidx = oracle.make_index(d, 3, 64, 8, cent, cb, offs, codes, ids)
    gidx = to_library(P, oidx)
    q = np.random.default_rng(810).standard_normal((6, d)).astype(np.float32)
    # (share: the one-pair kernel, the library's choice, and the group kernel with two and four pairs per workgroup)
    for share in (1, 0, 2, 4):
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, share)
        for probes_row, k in (([0, 1], 100), ([0, 1, 2], 1000), ([2, 1], 10), ([1, 2, 0], 10)):
            probes = np.tile(np.array([probes_row], dtype=np.uint32), (6, 1))
            for dtype in (oracle.LUT_FP32, oracle.LUT_E5M3):
                _step(f"split scan, everything in the race: share={share} probes={probes_row} k={k} dtype={dtype}: "
                      f"{gidx.ivfpq_scan_kernel_info(dtype)}")
                ids_g, d_g = gidx.ivfpq_search_with_probes(q, probes, k, dtype)
                ids_o, d_o = oracle.search(oidx, q, len(probes_row), k, dtype, probes=probes)
                assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context=f"share={share} probes={probes_row} k={k}")
    gidx.ivfpq_set_tuning(P.TUNE_SCAN_SHARE, 0)


@pytest.mark.usefixtures("route")
def test_search_nearest_cluster_smaller_than_k(P):
    # the cluster nearest to these queries holds 5 vectors, fewer than k: the search takes its bound from the
    # next probe that holds at least k (and scans that one unfiltered); the answer is the oracle's all the same
    n, d = 6000, 32
    cent, cb, _, codes, ids = si.random_index_arrays(n, d, 5, 16, 8, salt=820)
    offs = np.array([0, 5, 8, 3000, 3000, 6000], dtype=np.int64)          # 5, 3, 2992, 0 and 3000 vectors
    oidx = oracle.make_index(d, 5, 16, 8, cent, cb, offs, codes, ids)
    gidx = to_library(P, oidx)
    rng = np.random.default_rng(820)
    q = (cent[0] + 0.05 * rng.standard_normal((40, d))).astype(np.float32)
    q[20:] = (cent[1] + 0.05 * rng.standard_normal((20, d))).astype(np.float32)
    for n_probes, k in ((5, 10), (2, 10), (3, 4), (5, 1000), (1, 10)):
        for dtype in (oracle.LUT_FP32, oracle.LUT_E5M3):
            _step(f"nearest cluster smaller than k: P={n_probes} k={k} dtype={dtype}")
            ids_g, d_g, ids_o, d_o = _search_both(gidx, oidx, q, n_probes, k, dtype)
            assert_topk_matches(ids_g, d_g, ids_o, d_o, context=f"tiny nearest cluster P={n_probes} k={k}")


# ---------------------------------------------------------------- the search inside a HIP graph

@pytest.mark.usefixtures("route")
def test_search_replays_correctly_from_a_hip_graph(P, tiny):
    # a serving loop may capture the search call once and replay it: the call only enqueues kernels
    # (no allocation, no synchronisation, no memset), so every replay must give the eager result
    w, data, oidx, gidx = tiny
    qs = si.queries(w, 192)
    q = torch.from_numpy(qs[:64]).cuda()
    out = (torch.empty((64, w.k), dtype=torch.int64, device="cuda"), torch.empty((64, w.k), dtype=torch.float32, device="cuda"))
    for dtype in (P.LUT_FP8_E5M3, P.LUT_FP32):
        _step(f"graph capture lut={dtype}")
        q.copy_(torch.from_numpy(qs[:64]))
        gidx.ivfpq_search(q, w.n_probes, w.k, dtype, out=out)          # eager: workspace and kernel attributes in place
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            gidx.ivfpq_search(q, w.n_probes, w.k, dtype, out=out)
        for rep in range(4):
            q.copy_(torch.from_numpy(qs[64 * (rep % 3):64 * (rep % 3) + 64]))      # new queries in the captured buffer
            want_i, want_d = gidx.ivfpq_search(q.clone(), w.n_probes, w.k, dtype)  # eager work between the replays
            torch.cuda.synchronize()
            out[0].fill_(-7)
            out[1].fill_(-1.0)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out[0], want_i) and torch.equal(out[1], want_d), f"replay {rep}"
        del g


@pytest.mark.usefixtures("route")
def test_workspace_limit_changes_tiling_not_results(P, tiny):
    w, data, oidx, gidx = tiny
    q = torch.from_numpy(si.queries(w, 300)).cuda()
    big = gidx.ivfpq_search_workspace_bytes(300, w.n_probes, w.k, P.LUT_FP8_E5M3)
    want = gidx.ivfpq_search(q, w.n_probes, w.k, P.LUT_FP8_E5M3)
    torch.cuda.synchronize()
    try:
        gidx.ivfpq_set_workspace_limit(1 << 20)             # a few queries per tile
        small = gidx.ivfpq_search_workspace_bytes(300, w.n_probes, w.k, P.LUT_FP8_E5M3)
        assert small < big
        _step(f"workspace limit 1 MiB: {small} bytes instead of {big}")
        got = gidx.ivfpq_search(q, w.n_probes, w.k, P.LUT_FP8_E5M3)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        with pytest.raises(P.IvfpqError):
            gidx.ivfpq_set_workspace_limit(1000)
    finally:
        gidx.ivfpq_set_workspace_limit(32 << 30)


# ---------------------------------------------------------------- seeded random configurations

@pytest.mark.usefixtures("route")
def test_search_seeded_random_configurations(P):
    # thirty configurations drawn from a seeded generator: code widths 4-8 bits, sub-vector lengths 1-6,
    # few or many clusters (some empty), any table dtype and encoding option, k and n_probes up to the
    # limits that the configuration allows
    rng = np.random.default_rng(20230106)
    for case in range(30):
        bits = int(rng.integers(4, 9))
        unit = {4: 8, 5: 32, 6: 16, 7: 32, 8: 4}[bits]             # sub-spaces per 32-bit boundary
        pq_dim = unit * int(rng.integers(1, 5 if unit < 32 else 3))
        m = int(rng.choice([1, 2, 3, 4, 6]))
        d = pq_dim * m
        n_lists = int(rng.choice([1, 2, 7, 33, 200, 1500]))
        n = int(rng.integers(max(n_lists, 50), 6000))
        empty = tuple(int(v) for v in rng.choice(n_lists, size=min(3, n_lists - 1), replace=False)) if n_lists > 3 else ()
        n_probes = int(rng.integers(1, min(n_lists, 40) + 1))
        k = int(rng.choice([1, 5, 10, 100, 1000]))
        dtype = int(rng.integers(0, 4))
        trunc, per_table = bool(rng.integers(0, 2)), bool(rng.integers(0, 2))
        scale = float(rng.choice([1e-3, 1.0, 30.0]))
        oidx, gidx = random_pair(P, n, d, n_lists, pq_dim, bits, salt=7000 + case, scale=scale, empty_lists=empty)
        q = (scale * rng.standard_normal((17, d))).astype(np.float32)
        kw = {}
        if dtype in FP8:
            bias = 15 if dtype == oracle.LUT_E5M3 else 7
            gidx.ivfpq_set_fp8_encoding(dtype, bias, int(trunc), per_table)
            kw = dict(truncate=trunc, bias=bias, per_table=per_table)
        _step(f"random case {case}: n={n} d={d} lists={n_lists} s={pq_dim} p={bits} P={n_probes} k={k} dtype={dtype} {kw}")
        ids_g, d_g = gidx.ivfpq_search(q, n_probes, k, dtype)
        probes, _ = gidx.ivfpq_select_probes(q, n_probes)
        probes = probes.cpu().numpy().view(np.uint32)
        assert_probes_match(probes, oidx.centroids, q, n_probes)
        ids_o, d_o = oracle.search(oidx, q, n_probes, k, dtype, probes=probes, **kw)
        assert_topk_matches(ids_g.cpu().numpy(), d_g.cpu().numpy(), ids_o, d_o, context=f"random case {case}")
        gidx.ivfpq_free()


@pytest.mark.usefixtures("route")
def test_search_index_without_vectors(P):
    # every cluster empty: nothing faults, every result slot is padding
    d, n_lists, pq_dim = 32, 12, 16
    rng = np.random.default_rng(77)
    cent = rng.standard_normal((n_lists, d)).astype(np.float32)
    cb = rng.standard_normal((pq_dim, 256, 2)).astype(np.float32)
    gidx = P.Index.ivfpq_index_from_arrays(d, n_lists, pq_dim, 8, cent, cb, np.zeros(n_lists + 1, np.int64),
                                           np.zeros((0, pq_dim), np.uint8), np.zeros(0, np.int64)).ivfpq_upload()
    q = rng.standard_normal((9, d)).astype(np.float32)
    for n_probes in (1, 5, 12):
        _step(f"empty index P={n_probes}")
        ids, dist = gidx.ivfpq_search(q, n_probes, 7, P.LUT_FP8_E5M3)
        assert (ids.cpu().numpy() == -1).all() and np.isinf(dist.cpu().numpy()).all()
    probes, _ = gidx.ivfpq_select_probes(q, 12)
    assert_probes_match(probes.cpu().numpy().view(np.uint32), cent, q, 12)


@pytest.mark.parametrize("n_lists", [65, 127, 256, 259, 1000, 1024, 1190])
def test_select_probes_by_waves(P, n_lists):
    # 1,537 queries and up to 64 probes of at most 2 strips a probe: a wave per query; 65 probes and 1,536 queries: a workgroup per query.  Rows
    # that are and are not whole 16-byte words, fewer and more clusters than the 256 minima, ties, more equal ranking values than a wave holds
    # candidates, a query that is no number.
    rng = np.random.default_rng(n_lists)
    d = 32
    cen = (rng.standard_normal((n_lists, d)) * 10).astype(np.float32)
    cen[1::7] = cen[0]                                       # exact ties
    if n_lists == 1000:
        cen[200:800] = cen[200]                              # a plateau: 600 candidates
    books = rng.standard_normal((16, 16, 2)).astype(np.float32)
    codes = rng.integers(0, 256, (n_lists, 8)).astype(np.uint8)
    oidx = oracle.make_index(d, n_lists, 16, 4, cen, books, np.arange(n_lists + 1, dtype=np.int64), codes, np.arange(n_lists, dtype=np.int64))
    gidx = to_library(P, oidx)
    q = (cen[rng.integers(0, n_lists, 1537)] + rng.standard_normal((1537, d))).astype(np.float32)
    q[7] = cen[0]
    some = np.r_[0:200, 1337:1537]
    for n_probes, nq in ((1, 1537), (20, 1537), (63, 1537), (64, 1537), (min(65, n_lists), 1537), (64, 1536)):
        _step(f"select_probes by waves L={n_lists} P={n_probes} nq={nq}")
        at = some[some < nq]
        probes, pd = (x.cpu().numpy()[at] for x in gidx.ivfpq_select_probes(q[:nq], n_probes))
        want_d = oracle.select_probes(oidx, q[at], n_probes)[1]
        assert_probes_match(probes.view(np.uint32), cen, q[at], n_probes)
        np.testing.assert_allclose(pd, want_d, rtol=RTOL)
        # ties go to the lower cluster, whichever path takes them
        assert np.all((np.diff(pd, axis=1) > 0) | (np.diff(probes.astype(np.int64), axis=1) > 0))
    q[9, 3] = np.nan
    probes = gidx.ivfpq_select_probes(q, 20)[0].cpu().numpy()
    others = some[some != 9]
    assert_probes_match(probes.view(np.uint32)[others], cen, q[others], 20)
    assert len(set(probes[9].tolist())) == 20


def _offset_probes(P, n_lists, d, offset, nq, seed):
    """Clusters and queries that all lie `offset` from the origin in every component: the ranking values' error bound goes with the norms."""
    rng = np.random.default_rng(seed)
    cen = (offset + 128.0 * rng.random((n_lists, d))).astype(np.float32)
    books = rng.standard_normal((16, 16, d // 16)).astype(np.float32)
    codes = rng.integers(0, 256, (n_lists, 8)).astype(np.uint8)
    gidx = to_library(P, oracle.make_index(d, n_lists, 16, 4, cen, books, np.arange(n_lists + 1, dtype=np.int64), codes, np.arange(n_lists, dtype=np.int64)))
    return cen, (cen[rng.integers(0, n_lists, nq)] + 20.0 * rng.standard_normal((nq, d))).astype(np.float32), gidx


@pytest.mark.parametrize("n_lists,d,offset", [(320, 32, 3000), (1024, 128, 700), (1024, 128, 2000), (1190, 64, 1500), (2002, 128, 500)])
def test_select_probes_of_vectors_that_share_an_offset(P, n_lists, d, offset):
    # more clusters within the error bound than a wave holds at a time (192), up to all of them: taken in rounds.  Exact all the same
    cen, q, gidx = _offset_probes(P, n_lists, d, offset, 2048, n_lists)
    some = np.arange(0, 2048, 43)
    dist = ((q[some, None, :].astype(np.float64) - cen[None].astype(np.float64)) ** 2).sum(-1)
    a = np.sort(dist, axis=1)                                # ranking values but for |q|^2
    slack = 2 * ((3 * d + 8) * 2.0 ** -22 + 5e-5) * ((q[some].astype(np.float64) ** 2).sum(1) + (cen.astype(np.float64) ** 2).sum(1).max())
    for n_probes in (1, 10, 63, 64):
        _step(f"select_probes at offset {offset}, L={n_lists} d={d} P={n_probes}")
        admitted = (a <= (a[:, n_probes - 1] + slack)[:, None]).sum(1)
        if n_probes == 64:
            assert np.median(admitted) > 192
        probes, pd = (x.cpu().numpy() for x in gidx.ivfpq_select_probes(q, n_probes))
        assert_probes_match(probes[some].view(np.uint32), cen, q[some], n_probes)
        np.testing.assert_allclose(pd[some], a[:, :n_probes], rtol=RTOL)
        assert np.all((np.diff(pd, axis=1) > 0) | (np.diff(probes.astype(np.int64), axis=1) > 0))


def test_an_offset_costs_the_selection_little(P):
    # 8,000 clusters, 64 probes, hundreds of candidates a query: not many times what as many queries of centred vectors take (0.11 ms; exact distances
    # of all clusters and then a pass over them for every probe took 36 times that)
    took = {}
    for offset in (0.0, 400.0):
        cen, q, gidx = _offset_probes(P, 8000, 128, offset, 4096, 5)
        q = torch.from_numpy(q).cuda()
        _step(f"time of select_probes at offset {offset}")
        runs = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            gidx.ivfpq_select_probes(q, 64)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b))
        took[offset] = min(runs)
    assert took[400.0] < 8 * took[0.0]


@pytest.mark.parametrize("n_lists,d", [(193, 32), (1000, 32), (1024, 128), (2000, 96), (4000, 32)])
def test_select_probes_by_waves_of_far_queries(P, n_lists, d):
    # centred clusters, few within each other's error bound, so that the selection goes by waves; queries so far out that all or hundreds of
    # them are within theirs (which goes with |q|^2): rounds of 192, beside queries that need none
    rng = np.random.default_rng(n_lists)
    cen = (10 * rng.standard_normal((n_lists, d))).astype(np.float32)
    books = rng.standard_normal((16, 16, d // 16)).astype(np.float32)
    gidx = to_library(P, oracle.make_index(d, n_lists, 16, 4, cen, books, np.arange(n_lists + 1, dtype=np.int64), rng.integers(0, 256, (n_lists, 8)).astype(np.uint8),
                                           np.arange(n_lists, dtype=np.int64)))
    q = (cen[rng.integers(0, n_lists, 1600)] + rng.standard_normal((1600, d))).astype(np.float32)
    for i, far in enumerate((30, 100, 300, 1000, 3000)):
        q[i::8] += np.float32(far)
    for n_probes in (1, 10, 63, 64):
        _step(f"select_probes by waves, far queries, L={n_lists} d={d} P={n_probes}")
        probes, pd = (x.cpu().numpy() for x in gidx.ivfpq_select_probes(q, n_probes))
        assert_probes_match(probes.view(np.uint32)[::5], cen, q[::5], n_probes)
        assert np.all((np.diff(pd, axis=1) > 0) | (np.diff(probes.astype(np.int64), axis=1) > 0))
        few, few_d = (x.cpu().numpy() for x in gidx.ivfpq_select_probes(q[:500], n_probes))           # few queries: all distances, by workgroups
        np.testing.assert_allclose(pd[:500], few_d, rtol=RTOL)


@pytest.mark.parametrize("d,pq_dim,pq_bits", [(64, 16, 8), (128, 32, 8), (96, 48, 8), (128, 64, 8), (128, 64, 4), (128, 64, 7), (128, 32, 5)])
def test_nearest_probes_by_groups(P, d, pq_dim, pq_bits):
    # 5,000 queries on 41 clusters: where the encoding takes groups at that size (12,000 queries, and which kernels run: below), their nearest probes
    # are scanned by the group kernel and bounded by a wave each with scan route 0; with a route named, a workgroup each.  Lists of 1,
    # 63, 64, 65, 2,047, 2,049 (a wave holds 2,048 values), and 6,000 vectors, an empty one, one of equal codes (more values under the bound
    # than a wave gathers); k up to and past what a wave takes; queries that are no numbers.  Same bits.
    rng = np.random.default_rng(1000 * d + 10 * pq_dim + pq_bits)
    sizes = np.array([0, 1, 63, 64, 65, 127, 128, 129, 2047, 2048, 2049, 6000] + [700 + 3 * i for i in range(29)])
    cent = (4 * rng.standard_normal((41, d))).astype(np.float32)
    books = (0.5 * rng.standard_normal((pq_dim, 1 << pq_bits, d // pq_dim))).astype(np.float32)
    n = int(sizes.sum())
    codes = rng.integers(0, 256, (n, pq_dim * pq_bits // 8)).astype(np.uint8)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    codes[offsets[30]:offsets[31]] = codes[offsets[30]]
    gidx = to_library(P, oracle.make_index(d, 41, pq_dim, pq_bits, cent, books, offsets, codes, rng.permutation(n).astype(np.int64)))
    q = (cent[rng.integers(0, 41, 5000)] + 0.5 * rng.standard_normal((5000, d))).astype(np.float32)
    q[5] = np.nan
    q[6, 0] = np.inf
    q[7] *= 1e20
    for dtype in (oracle.LUT_FP32, oracle.LUT_FP16, oracle.LUT_E5M3, oracle.LUT_E4M4):
        for k in (1, 10, 100, 128, 129):
            out = []
            for route in (0, 3):
                gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
                _step(f"nearest probes by groups d={d} sub={pq_dim} bits={pq_bits} dtype={dtype} k={k} route={route}")
                out.append([t.cpu().numpy() for t in gidx.ivfpq_search(q, 12, k, dtype)])
            np.testing.assert_array_equal(out[0][0], out[1][0])
            np.testing.assert_array_equal(out[0][1].view(np.uint32), out[1][1].view(np.uint32))


@pytest.mark.parametrize("d,pq_dim,pq_bits", [(96, 96, 5), (96, 96, 6), (64, 64, 8)])
def test_nearest_probes_by_groups_round_as_one_query_does(P, d, pq_dim, pq_bits):
    # One-component sub-vectors have entries over the formats' whole range, so that sums are rounded: the group kernel's are the ones that a
    # workgroup a query forms, to the last bit.  (The filter is kept out of both: the other probes go the same way.)
    rng = np.random.default_rng(pq_bits)
    cent = (4 * rng.standard_normal((40, d))).astype(np.float32)
    books = (0.5 * rng.standard_normal((pq_dim, 1 << pq_bits, 1))).astype(np.float32)
    codes = rng.integers(0, 256, (40_000, pq_dim * pq_bits // 8)).astype(np.uint8)
    gidx = to_library(P, oracle.make_index(d, 40, pq_dim, pq_bits, cent, books, np.arange(41, dtype=np.int64) * 1000, codes, np.arange(40_000, dtype=np.int64)))
    gidx.ivfpq_set_tuning(P.TUNE_EARLY_EXIT, -1)
    q = torch.from_numpy((cent[rng.integers(0, 40, 12_000)] + 30 * rng.standard_normal((12_000, d))).astype(np.float32)).cuda()
    for dtype in (oracle.LUT_E5M3, oracle.LUT_E4M4):
        out = []
        for route in (0, 3):
            gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
            _step(f"rounding of nearest probes by groups d={d} bits={pq_bits} dtype={dtype} route={route}")
            out.append([t.cpu().numpy() for t in gidx.ivfpq_search(q, 2, 128, dtype)])
        np.testing.assert_array_equal(out[0][1].view(np.uint32), out[1][1].view(np.uint32))
        np.testing.assert_array_equal(out[0][0], out[1][0])


def _bound_ms(P, gidx):
    # the launch that bounds the nearest probes scanned by groups; 0: a workgroup a query has scanned and bounded them
    ms = (ctypes.c_float * 8)()
    assert P.lib().ivfpq_stage_times_ms(gidx._h, ctypes.byref(ms)) == 0
    assert 0 <= ms[7] <= ms[5] <= ms[1]
    return ms[7]


def _both_routes(P, gidx, q, n_probes, k, dtype, grouped, context):
    # route 0 against a workgroup a query (any route named): the same bits; by the stage times, which of them has run.  The other probes go the
    # same way in both, since the tables' sums are rounded in another order than the filter's candidates: a route named means the
    # filter, which the knob of the early exit keeps out.
    out = []
    for route in (0, 3):
        _step(f"{context} k={k} dtype={dtype} route={route}")
        gidx.ivfpq_set_tuning(P.TUNE_SCAN_ROUTE, route)
        gidx.ivfpq_set_stage_timing(True)
        out.append([t.cpu().numpy() for t in gidx.ivfpq_search(q, n_probes, k, dtype)])
        name = gidx.ivfpq_scan_kernel_info(dtype).split("<")[0]
        assert (_bound_ms(P, gidx) > 0) == (grouped and route == 0), f"{context} k={k} dtype={dtype} route={route}"
        gidx.ivfpq_set_stage_timing(False)
        gidx.ivfpq_set_tuning(P.TUNE_EARLY_EXIT, -1 if route == 0 and name != "scan_filter_kernel" else 0)
        others = name if route == 0 else others
        assert name == others
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1].view(np.uint32), out[1][1].view(np.uint32))
    return out[0]


@pytest.mark.parametrize("d,pq_dim,pq_bits,few", [
    (64, 16, 8, ""), (128, 32, 8, ""), (96, 48, 8, "4"), (128, 64, 8, "4"), (64, 64, 8, "42"), (96, 96, 7, "42"), (96, 96, 6, "4"), (96, 96, 5, ""),
    (96, 48, 6, ""), (128, 64, 7, ""), (64, 32, 7, "2"), (64, 32, 5, "2"), (128, 64, 4, "1"), (128, 32, 4, "41"), (96, 96, 4, "1"), (64, 64, 4, "1")])
def test_nearest_probes_of_every_encoding_by_groups(P, d, pq_dim, pq_bits, few):
    # 12,000 queries on 43 clusters.  few: tables (bytes an entry) that take a workgroup a query, too large for two of them or never faster in
    # groups; of the others the group kernel is seen to run.  Lists of 0 to 6,000 vectors, one of equal codes, queries that are no numbers.
    rng = np.random.default_rng(1000 * d + 10 * pq_dim + pq_bits)
    sizes = np.array([0, 1, 63, 64, 65, 127, 128, 129, 2047, 2048, 2049, 6000] + [900 + 3 * i for i in range(31)])
    cent = (4 * rng.standard_normal((43, d))).astype(np.float32)
    books = (0.5 * rng.standard_normal((pq_dim, 1 << pq_bits, d // pq_dim))).astype(np.float32)
    n = int(sizes.sum())
    codes = rng.integers(0, 256, (n, pq_dim * pq_bits // 8)).astype(np.uint8)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    codes[offsets[30]:offsets[31]] = codes[offsets[30]]
    oidx = oracle.make_index(d, 43, pq_dim, pq_bits, cent, books, offsets, codes, rng.permutation(n).astype(np.int64))
    gidx = to_library(P, oidx)
    q = (cent[rng.integers(0, 43, 12_000)] + 0.5 * rng.standard_normal((12_000, d))).astype(np.float32)
    q[5] = np.nan
    q[6, 0] = np.inf
    q[7] *= 1e20
    q = torch.from_numpy(q).cuda()
    for dtype, size in ((oracle.LUT_FP32, "4"), (oracle.LUT_FP16, "2"), (oracle.LUT_E5M3, "1"), (oracle.LUT_E4M4, "1")):
        for k in (1, 100, 128, 129):
            ids, dist = _both_routes(P, gidx, q, 12, k, dtype, size not in few and k <= 128, f"nearest by groups d={d} sub={pq_dim} bits={pq_bits}")
            if dtype == oracle.LUT_FP32 and k == 100:
                at = rng.integers(8, 12_000, 24)
                want_ids, want_d = oracle.search(oidx, q[at].cpu().numpy(), 12, k)
                assert_topk_matches(ids[at], dist[at], want_ids, want_d, context=f"d={d} sub={pq_dim} bits={pq_bits}")


@pytest.mark.parametrize("dtype", DTYPES)
def test_nearest_probes_by_groups_without_a_bound(P, dtype):
    # every probed list is shorter than k, some are empty, so that no value bounds anything: all vectors are admitted; with k small
    # enough, only by the queries whose probes are all shorter
    rng = np.random.default_rng(int(dtype) + 5)
    sizes = rng.integers(40, 100, 80)
    sizes[::9] = 0
    sizes[1::9] = 1
    d, pq_dim = 128, 32
    cent = (4 * rng.standard_normal((80, d))).astype(np.float32)
    books = (0.5 * rng.standard_normal((pq_dim, 256, 4))).astype(np.float32)
    n = int(sizes.sum())
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    oidx = oracle.make_index(d, 80, pq_dim, 8, cent, books, offsets, rng.integers(0, 256, (n, pq_dim)).astype(np.uint8), rng.permutation(n).astype(np.int64))
    gidx = to_library(P, oidx)
    q = (cent[rng.integers(0, 80, 9_000)] + 0.5 * rng.standard_normal((9_000, d))).astype(np.float32)
    for k in (60, 100, 128):
        ids, dist = _both_routes(P, gidx, torch.from_numpy(q).cuda(), 20, k, dtype, True, "nearest by groups, short lists")
        if dtype == oracle.LUT_FP32:
            at = rng.integers(0, 9_000, 32)
            want_ids, want_d = oracle.search(oidx, q[at], 20, k)
            assert_topk_matches(ids[at], dist[at], want_ids, want_d, context=f"k={k}")


def test_nearest_probes_by_groups_subnormal(P):
    # distances below the least normal number, and a list that has fewer than k of them above zero
    rng = np.random.default_rng(9)
    d, pq_dim, lists = 128, 32, 30
    tiny = np.float32(2e-21)
    cent = (8 * rng.standard_normal((lists, d))).astype(np.float32) * tiny
    books = rng.standard_normal((pq_dim, 256, 4)).astype(np.float32) * tiny
    n = lists * 900
    offsets = np.arange(lists + 1, dtype=np.int64) * 900
    oidx = oracle.make_index(d, lists, pq_dim, 8, cent, books, offsets, rng.integers(0, 256, (n, pq_dim)).astype(np.uint8), np.arange(n, dtype=np.int64))
    gidx = to_library(P, oidx)
    q = (cent[rng.integers(0, lists, 8_000)] + rng.standard_normal((8_000, d)).astype(np.float32) * tiny).astype(np.float32)
    for k in (10, 100):
        ids, dist = _both_routes(P, gidx, torch.from_numpy(q).cuda(), 15, k, oracle.LUT_FP32, True, "nearest by groups, subnormal")
        assert 0 < dist.max() < np.finfo(np.float32).tiny


def test_nearest_probes_by_groups_tile_by_tile(P):
    # tiles of which the last is too small for groups, and a batch that one launch cannot order: the results of a workgroup a query
    rng = np.random.default_rng(4)
    d, pq_dim, lists = 128, 64, 40
    cent = (4 * rng.standard_normal((lists, d))).astype(np.float32)
    books = (0.5 * rng.standard_normal((pq_dim, 256, 2))).astype(np.float32)
    n = lists * 800
    offsets = np.arange(lists + 1, dtype=np.int64) * 800
    gidx = to_library(P, oracle.make_index(d, lists, pq_dim, 8, cent, books, offsets, rng.integers(0, 256, (n, pq_dim)).astype(np.uint8), np.arange(n, dtype=np.int64)))
    q = torch.from_numpy((cent[rng.integers(0, lists, 16_385)] + 0.5 * rng.standard_normal((16_385, d))).astype(np.float32)).cuda()
    whole = _both_routes(P, gidx, q[:16_384].contiguous(), 15, 10, oracle.LUT_E5M3, True, "16,384 queries")
    _both_routes(P, gidx, q, 15, 10, oracle.LUT_E5M3, False, "16,385 queries")
    need = gidx.ivfpq_search_workspace_bytes(8_000, 15, 10, oracle.LUT_E5M3)
    gidx.ivfpq_set_workspace_limit(need)                     # 16,384 queries: two tiles of about 8,000 and a small one, or nearly so
    parts = _both_routes(P, gidx, q[:16_384].contiguous(), 15, 10, oracle.LUT_E5M3, True, "16,384 queries in tiles")
    np.testing.assert_array_equal(whole[0], parts[0])
    np.testing.assert_array_equal(whole[1].view(np.uint32), parts[1].view(np.uint32))
    _both_routes(P, gidx, q[:2_400].contiguous(), 15, 10, oracle.LUT_E5M3, False, "2,400 queries")
