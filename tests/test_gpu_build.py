"""GPU parity of the index construction (Sec. I-C, first enumeration) against the oracle's builder.

Both sides take every decision as the arg-min of float64 squared distances (ties to the lower index)
and form every centre as the float64 mean of its members in ascending row order, so with the same
training rows and the same k-means start rows the saved index must be IDENTICAL: centroids and
codebooks bit for bit, list offsets, ids and packed codes byte for byte.
"""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2301_06672_amd as pkg
    pkg.lib()
    assert torch.cuda.is_available()
    return pkg


def _step(msg):
    print(f"[build] {msg}", flush=True)


def _data(n, d, seed, offset=0.0, kind="gauss"):
    rng = np.random.default_rng(seed)
    if kind == "intgrid":           # integer-valued components: plenty of exactly equal distances
        return rng.integers(0, 6, size=(n, d)).astype(np.float32)
    centres = rng.standard_normal((12, d)) * 2.0
    x = centres[rng.integers(0, 12, size=n)] + 0.7 * rng.standard_normal((n, d))
    return (x + offset).astype(np.float32)


# ---------------------------------------------------------------- the assignment step alone

@pytest.mark.parametrize("n,d,k,offset,kind", [(5000, 48, 300, 0.0, "gauss"), (3000, 32, 64, 500.0, "gauss"),
                                               (4000, 16, 200, 0.0, "intgrid"), (1000, 7, 3, 0.0, "gauss"),
                                               (700, 128, 1, 0.0, "gauss"),
                                               # 256 centres or more: decided from strip summaries of the ranking values
                                               (20000, 32, 2000, 0.0, "gauss"),      # 128 x 128 bf16 tiles, 64-centre strips
                                               (6000, 16, 700, 0.0, "intgrid"),      # ties, ragged last 32-centre strip
                                               (5000, 24, 1000, 500.0, "gauss"),     # most rows through the float64 path
                                               (40000, 8, 4000, 0.0, "intgrid"),     # ties under the bf16 tiles
                                               (30000, 20, 3000, 0.0, "gauss")])     # d not a multiple of the bf16 slices
def test_assign_device_equals_oracle(P, n, d, k, offset, kind):
    # offset 500: norms dwarf the distances, so many rows go through the exact float64 path;
    # intgrid: exactly tied distances, decided by the lower index
    x = _data(n, d, 11 + n, offset, kind)
    rng = np.random.default_rng(5 + k)
    c = x[np.sort(rng.choice(n, size=k, replace=False))].copy()
    if k >= 8:
        c[5] = c[2]                  # a duplicated centre: the lower index must win
        c[7] = x[0]
    _step(f"assign n={n} d={d} k={k} offset={offset} {kind}")
    got = P.ivfpq_assign_device(x, c).cpu().numpy()
    want, _ = oracle.assign(x, c)
    np.testing.assert_array_equal(got, want)
    if k >= 8:
        assert not np.any(got == 5)


@pytest.mark.parametrize("n,d,k,kind", [
    (12001, 128, 1000, "gauss"),      # three blocks of rows per wave, a last tile of one row, a last stage of 40 centres
    (9000, 96, 1345, "gauss"),        # splits of the centres among workgroups; one centre past a stage
    (50000, 33, 257, "gauss"),        # two slices padded from 33 components
    (8000, 64, 1600, "offset"),       # a common offset of 1000 sigma: the mean comes off before the rounding to half
    (7000, 24, 2000, "same"),         # 60 copies of one centre: more centres within the bound than a row's list holds
    (6500, 16, 2048, "scales"),       # rows 10^6 times the centres' size and 10^-6 of it; components past the range of a half
    (9000, 100, 1400, "tiny"),        # values about 1e-30
])
def test_assign_device_half_precision_product(P, n, d, k, kind):
    # one product in half precision decides where the margin is larger than twice its error; the others are listed and compared in
    # float64: the oracle's labels, always
    rng = np.random.default_rng(n + d)
    x = _data(n, d, 31 + n, 1000.0 if kind == "offset" else 0.0, "gauss")
    if kind == "tiny":
        x *= np.float32(1e-30)
    c = x[np.sort(rng.choice(n, size=k, replace=False))].copy()
    c += (rng.standard_normal(c.shape) * 0.05 * x.std()).astype(np.float32)
    if kind == "same":
        c[700:760] = c[3]
        x[100:400] = c[3] + (rng.standard_normal((300, d)) * 0.01).astype(np.float32)
    if kind == "scales":
        x[::7] *= np.float32(1e6)
        x[1::7] *= np.float32(1e-6)
    c[11] = c[4]
    assert n * k >= 12_000_000                # what this way of deciding is taken from
    _step(f"assign, half-precision product: n={n} d={d} k={k} {kind}")
    got = P.ivfpq_assign_device(x, c).cpu().numpy()
    want, _ = oracle.assign(x, c)
    np.testing.assert_array_equal(got, want)
    if kind == "gauss":
        x[5, 2], x[n - 1, 0] = np.nan, np.inf                      # no nearest centre: a label in range, the other rows as before
        c2 = c.copy()
        c2[20, 3] = np.nan                                         # never the nearest
        got = P.ivfpq_assign_device(x, c2).cpu().numpy()
        want, _ = oracle.assign(x, c2)
        ok = np.ones(n, bool)
        ok[[5, n - 1]] = False
        np.testing.assert_array_equal(got[ok], want[ok])
        assert 0 <= got[5] < k and 0 <= got[n - 1] < k and not np.any(got == 20)


@pytest.mark.parametrize("d", [16, 128])
def test_assign_device_half_precision_product_centres_past_its_range(P, d):
    # finite centres whose components are so large that their squares leave a float's range are no part of the half-precision
    # product, and still the nearest of the rows around them
    n, k = 9000, 1500
    rng = np.random.default_rng(d)
    c = (rng.uniform(-9e17, 9e17, (k, d))).astype(np.float32)
    c[[7, 640, 1499]] = rng.uniform(1.5e18, 2.5e18, (3, d)).astype(np.float32)
    at = rng.integers(0, k, n)
    at[::50] = 640
    x = (c[at] + rng.uniform(-1e17, 1e17, (n, d))).astype(np.float32)
    _step(f"assign, centres on both sides of 1e18: d={d}")
    got = P.ivfpq_assign_device(x, c).cpu().numpy()
    want, _ = oracle.assign(x, c)
    assert np.mean(want == 640) > 0.015
    np.testing.assert_array_equal(got, want)


# ---------------------------------------------------------------- the whole build

def _rows(n, n_lists, pq_dim, pq_bits, n_ct, n_pt, salt):
    ct = si.stride_sample(n, n_ct)
    pt = si.stride_sample(n, n_pt)
    ci = si.kmeans_init_rows(si.STREAM_COARSE_INIT, 0, len(ct), n_lists, salt)
    pi = np.stack([si.kmeans_init_rows(si.STREAM_PQ_INIT, j, len(pt), 1 << pq_bits, salt) for j in range(pq_dim)])
    return ct, ci, pt, pi


def _assert_same_index(gidx, oidx):
    cent, cb, offs, codes, ids = gidx.ivfpq_index_export()
    np.testing.assert_array_equal(offs, oidx.list_offsets)
    np.testing.assert_array_equal(ids, oidx.ids)
    np.testing.assert_array_equal(cent.view(np.uint32), oidx.centroids.view(np.uint32))
    np.testing.assert_array_equal(cb.view(np.uint32).reshape(-1), oidx.codebooks.view(np.uint32).reshape(-1))
    np.testing.assert_array_equal(codes.reshape(oidx.codes.shape), oidx.codes)


@pytest.mark.parametrize("n,d,n_lists,pq_dim,pq_bits,iters,n_ct,n_pt,kind", [
    (10_000, 32, 64, 16, 8, 4, 5_000, 4_000, "gauss"),      # m = 2
    (6_000, 24, 20, 8, 4, 3, 6_000, 6_000, "gauss"),        # 4-bit codes, m = 3, all rows train
    (6_000, 64, 16, 8, 8, 3, 3_000, 2_500, "gauss"),        # m = 8: the generic sub-vector path
    (20_000, 16, 2, 16, 8, 2, 20_000, 3_000, "gauss"),      # two huge lists: groups longer than one LDS sort
    (5_000, 32, 40, 32, 8, 3, 2_500, 2_000, "intgrid"),     # m = 1, tied distances everywhere
    (3_000, 32, 48, 16, 8, 0, 1_000, 1_000, "gauss"),       # no Lloyd iteration: the start rows are the centres
    (4_000, 64, 12, 32, 5, 2, 4_000, 2_000, "gauss"),       # 5-bit codes: 32 sub-spaces in 5 words
    (4_000, 32, 12, 16, 6, 2, 2_000, 2_000, "gauss"),       # 6-bit codes: 16 sub-spaces in 3 words
    (4_000, 64, 12, 32, 7, 2, 4_000, 2_000, "intgrid"),     # 7-bit codes, tied distances
    (30_000, 32, 512, 16, 8, 3, 15_000, 4_000, "gauss"),    # 512 lists: nearest centres from strip summaries
])
def test_build_device_is_identical_to_oracle_build(P, n, d, n_lists, pq_dim, pq_bits, iters, n_ct, n_pt, kind):
    x = _data(n, d, 100 + n + d, 0.0, kind)
    ct, ci, pt, pi = _rows(n, n_lists, pq_dim, pq_bits, n_ct, n_pt, salt=n + d)
    _step(f"build n={n} d={d} lists={n_lists} s={pq_dim} p={pq_bits} iters={iters} {kind}")
    gidx = P.Index.ivfpq_build_device(x, n_lists, pq_dim, pq_bits, iters, coarse_train_rows=ct, coarse_init_rows=ci,
                                      pq_train_rows=pt, pq_init_rows=pi)
    oidx = oracle.build_index(x, n_lists, pq_dim, pq_bits, iters, ci, pi, coarse_train_rows=ct, pq_train_rows=pt)
    _assert_same_index(gidx, oidx)


def test_more_lists_than_group_counters_fit(P):
    # above 32,768 lists the rows are grouped by atomics and sorted; one list holds far more than one sort takes in LDS
    n, d, n_lists = 42_000, 8, 32_800
    x = _data(n, d, 77)
    x[3::4] = x[3]
    ct = np.arange(n_lists)
    pt = np.arange(1000)
    pi = np.tile(np.arange(16) * 60, (8, 1))
    _step(f"build n={n} lists={n_lists}")
    gidx = P.Index.ivfpq_build_device(x, n_lists, 8, 4, 0, coarse_train_rows=ct, coarse_init_rows=ct, pq_train_rows=pt, pq_init_rows=pi)
    oidx = oracle.build_index(x, n_lists, 8, 4, 0, ct, pi, coarse_train_rows=ct, pq_train_rows=pt)
    assert np.diff(oidx.list_offsets).max() > 2 * 4096
    _assert_same_index(gidx, oidx)


@pytest.mark.parametrize("m,pq_bits", [(2, 8), (4, 8), (8, 8), (4, 7), (8, 7), (2, 6), (4, 6), (8, 6), (2, 5), (4, 5), (8, 5)])
@pytest.mark.parametrize("n,kind", [(255, "intgrid"), (513, "gauss"), (4097, "huge"), (1500, "offset")])
def test_codes_on_the_matrix_cores(P, m, pq_bits, n, kind):
    # workgroups of 512 positions, ragged at both ends; tied codewords (intgrid, and more codewords than distinct
    # rows); magnitudes whose squares overflow fp32, so that every codeword is compared in float64 (huge); residuals
    # that are small beside their codewords' error bound (offset: one list, far from the rows' mean)
    pq_dim = 32 if pq_bits in (5, 7) else 16
    d, n_lists = pq_dim * m, 1 if kind == "offset" else 4
    x = _data(n, d, 7 * n + m, 0.0, "intgrid" if kind == "intgrid" else "gauss")
    if kind == "huge":
        x = (x * np.float32(4e18)).astype(np.float32)
    if kind == "offset":
        x[::2] += 300.0
    n_t = min(n, 700)
    ct, ci, pt, pi = _rows(n, n_lists, pq_dim, pq_bits, n_t, n_t, salt=n + d) if n_t >= (1 << pq_bits) else (None,) * 4
    if ct is None:
        ct = pt = np.arange(n)
        ci = np.arange(n_lists) * (n // n_lists)
        pi = np.tile(np.arange(1 << pq_bits) % n, (pq_dim, 1))      # the same row twice: equal codewords
    _step(f"codes n={n} m={m} p={pq_bits} {kind}")
    gidx = P.Index.ivfpq_build_device(x, n_lists, pq_dim, pq_bits, 2, coarse_train_rows=ct, coarse_init_rows=ci,
                                      pq_train_rows=pt, pq_init_rows=pi)
    oidx = oracle.build_index(x, n_lists, pq_dim, pq_bits, 2, ci, pi, coarse_train_rows=ct, pq_train_rows=pt)
    _assert_same_index(gidx, oidx)


def test_build_device_default_draws_and_search(P):
    # rows drawn from the seed inside the library: a valid index that searches as well as the host-built one
    w = si.WORKLOADS["tiny"]
    data, q = si.dataset(w), si.queries(w, 200)
    _step("build_device (seeded draws) + search")
    g = P.Index.ivfpq_build_device(data, w.n_lists, w.pq_dim, w.pq_bits, 6, seed=3)
    g2 = P.Index.ivfpq_build_device(torch.from_numpy(data).cuda(), w.n_lists, w.pq_dim, w.pq_bits, 6, seed=3)
    for a, b in zip(g.ivfpq_index_export(), g2.ivfpq_index_export()):
        np.testing.assert_array_equal(a, b)                                   # deterministic
    cent, cb, offs, codes, ids = g.ivfpq_index_export()
    assert offs[0] == 0 and offs[-1] == w.n and np.all(np.diff(offs) >= 0)
    assert np.array_equal(np.sort(ids), np.arange(w.n))
    labels, _ = oracle.assign(data, cent)
    for l in range(w.n_lists):
        seg = ids[offs[l]:offs[l + 1]]
        assert np.all(np.diff(seg) > 0) and np.all(labels[seg] == l)
    gt, _ = oracle.exact_knn(data, q, w.k)
    h = P.Index.ivfpq_build_host(data, w.n_lists, w.pq_dim, w.pq_bits, 6, seed=3)
    rec = {}
    for name, idx in (("device", g), ("host", h)):
        idx.ivfpq_upload()
        found, _ = idx.ivfpq_search(q, w.n_probes, w.k, P.LUT_FP32)
        rec[name] = oracle.recall(found.cpu().numpy(), gt)
    _step(f"recall {rec}")
    assert abs(rec["device"] - rec["host"]) < 0.05 and rec["device"] > 0.5


@pytest.mark.parametrize("n", [5001, 800001])    # copied out by the runtime; by pieces through the pinned ring, the last one ragged
def test_build_device_arrays_arrive_whole(P, n):
    d, n_lists, pq_dim, bits = 16, 40, 16, 4
    x = _data(n, d, 5)
    _step(f"build_device n={n}, every id and code checked")
    cent, books, offs, codes, ids = P.Index.ivfpq_build_device(x, n_lists, pq_dim, bits, 1, seed=2).ivfpq_index_export()
    assert np.array_equal(np.sort(ids), np.arange(n))
    lists = np.repeat(np.arange(n_lists), np.diff(offs))
    assert np.all((np.diff(ids) > 0) | (np.diff(lists) > 0))
    word = np.stack([codes & 15, codes >> 4], axis=2).reshape(n, pq_dim)
    for j in range(pq_dim):                      # one component each: |residual - word| is the least there is, ties and rounding aside
        r = (x[ids, j] - cent[lists, j]).astype(np.float64)
        gap = np.abs(r[:, None] - books[j, :, 0].astype(np.float64))
        assert np.all(gap[np.arange(n), word[:, j]] <= gap.min(axis=1) + 1e-12)


def test_build_device_rejects_bad_arguments(P):
    x = torch.zeros((100, 16), device="cuda")
    for kw, status in ((dict(coarse_init_rows=np.full(4, 100)), P.EINVAL),
                       (dict(pq_train_rows=np.array([0, 5, 100])), P.EINVAL),
                       (dict(coarse_train_rows=np.array([-1, 2, 3, 4])), P.EINVAL)):
        with pytest.raises(P.IvfpqError) as e:
            P.Index.ivfpq_build_device(x, 4, 4, 8, 1, **kw)
        assert e.value.status == status
    with pytest.raises(P.IvfpqError):
        P.Index.ivfpq_build_device(x, 200, 4, 8, 1)          # more lists than rows
