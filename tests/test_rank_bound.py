"""CPU checks of the arithmetic behind probe selection's ranking values (no GPU, no library call):
the bf16 split of fp32 operands and the error bound that the kernels attach to a = |c|^2 - 2 q.c.
The kernels short-list with a() and decide with exact distances; these tests pin the claim that the
short list cannot miss a cluster, i.e. that the bound really bounds the error of the emulated arithmetic."""
import numpy as np
import pytest


def bf16_round(x):
    """fp32 -> nearest bf16 (ties to even), returned as fp32 with the low 16 bits clear."""
    b = np.asarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    r = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16) << 16
    return r.astype(np.uint32).view(np.float32)


def split(x):
    hi = bf16_round(x)
    rest = (x - hi).astype(np.float32)
    assert np.array_equal(rest.astype(np.float64), x.astype(np.float64) - hi.astype(np.float64))   # exact in fp32
    return hi, bf16_round(rest)


def rank_error_bound(d, qn, cmax):
    return ((3 * d + 8) * 2.0 ** -22 + 5.0e-5) * (qn + cmax)


def _cases():
    rng = np.random.default_rng(20230117)
    yield "integer grid", rng.integers(0, 256, size=(40, 128)).astype(np.float32), rng.integers(0, 256, size=(300, 128)).astype(np.float32)
    u = rng.standard_normal((40, 96)); v = rng.standard_normal((300, 96))
    yield "unit norm", (u / np.linalg.norm(u, axis=1, keepdims=True)).astype(np.float32), (v / np.linalg.norm(v, axis=1, keepdims=True)).astype(np.float32)
    yield "mixed scales", (rng.standard_normal((40, 64)) * 10.0 ** rng.integers(-6, 6, size=(1, 64))).astype(np.float32), \
        (rng.standard_normal((300, 64)) * 10.0 ** rng.integers(-6, 6, size=(1, 64))).astype(np.float32)
    yield "far from the origin", (1000.0 + rng.standard_normal((40, 32))).astype(np.float32), (1000.0 + rng.standard_normal((300, 32))).astype(np.float32)


@pytest.mark.parametrize("name,q,c", list(_cases()), ids=[n for n, _, _ in _cases()])
def test_split_remainder_is_within_its_bound(name, q, c):
    qh, ql = split(q)
    ch, cl = split(c)
    for x, h, l in ((q, qh, ql), (c, ch, cl)):
        assert np.all(np.abs(x.astype(np.float64) - h - l) <= 2.0 ** -16 * np.abs(x))
    f = np.float64
    exact = q.astype(f) @ c.astype(f).T
    kept = qh.astype(f) @ ch.astype(f).T + qh.astype(f) @ cl.astype(f).T + ql.astype(f) @ ch.astype(f).T
    mags = np.abs(q).astype(f) @ np.abs(c).astype(f).T
    assert np.all(np.abs(exact - kept) <= 3.02 * 2.0 ** -16 * mags)


@pytest.mark.parametrize("name,q,c", list(_cases()), ids=[n for n, _, _ in _cases()])
def test_emulated_ranking_value_stays_inside_the_bound(name, q, c):
    # fp32 accumulation of the 3 d exact products in a scrambled order, fp32 norm, fp32 multiply-add
    rng = np.random.default_rng(7)
    qh, ql = split(q)
    ch, cl = split(c)
    d = q.shape[1]
    cn = np.zeros(len(c), dtype=np.float32)
    for t in range(d):
        cn = (c[:, t] * c[:, t] + cn).astype(np.float32)
    cmax = float(cn.max())
    exact_a = (c.astype(np.float64) ** 2).sum(1)[None, :] - 2.0 * (q.astype(np.float64) @ c.astype(np.float64).T)
    terms = np.concatenate([qh[:, None, :] * ch[None, :, :], qh[:, None, :] * cl[None, :, :], ql[:, None, :] * ch[None, :, :]], axis=2)
    assert terms.dtype == np.float32        # bf16 x bf16 is exact in fp32
    order = rng.permutation(3 * d)
    acc = np.zeros(terms.shape[:2], dtype=np.float32)
    for t in order:
        acc = (acc + terms[:, :, t]).astype(np.float32)
    a = (np.float32(-2.0) * acc + cn[None, :]).astype(np.float32)
    qn = (q.astype(np.float64) ** 2).sum(1)
    delta = rank_error_bound(d, qn, cmax)[:, None]
    worst = np.max(np.abs(a.astype(np.float64) - exact_a) / delta)
    assert worst <= 0.5, f"{name}: error reaches {worst:.3f} of the bound"


def test_tagged_key_brackets_the_key():
    rng = np.random.default_rng(3)
    f = np.concatenate([rng.standard_normal(1000) * 1e3, -np.abs(rng.standard_normal(1000)), [0.0, -0.0]]).astype(np.float32)
    b = f.view(np.uint32)
    key = b ^ np.where(b >> 31, np.uint32(0xFFFFFFFF), np.uint32(0x80000000))
    order = np.argsort(key, kind="stable")
    assert np.all(np.diff(f[order]) >= 0)                          # the key map is monotone
    for col in (0, 17, 63):
        tagged = (key & np.uint32(0xFFFFFFC0)) | np.uint32(col)
        assert np.all((tagged & np.uint32(0xFFFFFFC0)) <= key) and np.all(key <= (tagged | np.uint32(63)))
        # what clearing six bits can lower a value by: 63 units in the last place, under 2^-17 of its magnitude
        # (or 63 denormal steps next to zero)
        lowered = (key & np.uint32(0xFFFFFFC0))
        back = lowered ^ np.where(lowered >> 31, np.uint32(0x80000000), np.uint32(0xFFFFFFFF))
        g = back.view(np.float32)
        ok = np.isfinite(g)
        assert np.all(g[ok] <= f[ok]) and np.all((f[ok].astype(np.float64) - g[ok]) <= 2.0 ** -17 * np.abs(f[ok]) + 64 * 2.0 ** -149)


# ---- the matrix-core filter of the grouped scan: a vector with R <= bound always passes its two tests

SHIM = r'''
#include "ivfpq_filter_bound.hpp"
using namespace ivfpq;
extern "C" void bound_of(int lut, int truncate, int pq_dim, int d, float* o) {
    const FilterBound b = filter_bound(lut, truncate != 0, pq_dim, d);
    const float v[13] = {b.scale, b.add, b.eta, kSquareLoss, kRoundedNorm, kEntrySlack, kHiddenSlack, kLimitShare, kWordNormSlack,
                         kCullNear, kCullRadius, kCullLimit, kCullTop};
    for (int i = 0; i < 13; ++i) o[i] = v[i];
}
'''
NAMES = ("scale add eta square_loss rounded_norm entry_slack hidden_slack limit_share word_norm_slack cull_near cull_radius "
         "cull_limit cull_top").split()


@pytest.fixture(scope="module")
def library_bound(tmp_path_factory):
    """The library's own numbers: its header, compiled on the spot."""
    import ctypes
    import os
    import subprocess
    where = tmp_path_factory.mktemp("bound")
    (where / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_06672_amd", "csrc")
    so = str(where / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, str(where / "shim.cpp"), "-o", so], check=True)
    shim = ctypes.CDLL(so)

    def of(dtype, truncate, subs, d):
        out = (ctypes.c_float * 13)()
        shim.bound_of(int(dtype), int(truncate), int(subs), int(d), out)
        return dict(zip(NAMES, [float(v) for v in out]))
    return of


def stored_entry(f, dtype, truncate=False):
    """A table entry as a lookup returns it: oracle dtypes 0 fp32, 1 half, 2 e5m3 (bias 15), 3 e4m4 (bias 1)."""
    if dtype == 0:
        return f
    if dtype == 1:
        return np.minimum(f, np.float32(65504.0)).astype(np.float16).astype(np.float32)
    shift, bias = (20, 15) if dtype == 2 else (19, 1)
    lo = (127 - bias) << 23
    b = np.clip(f.view(np.int32).astype(np.int64), lo, lo + (255 << shift))
    b = (b + (0 if truncate else 1 << (shift - 1))) & ~((1 << shift) - 1)
    return np.minimum(b, lo + (255 << shift)).astype(np.int32).view(np.float32)


TOP = {0: np.inf, 1: 65504.0, 2: 122880.0, 3: 1.9375 * 2.0 ** 14}         # oracle dtypes, as in stored_entry


def filter_margins(r, y, dtype, truncate, m, B, rng):
    """The kernel's arithmetic for one residual r and the decoded residuals y, with the numbers B: residuals and codewords in bf16, the
    product and its start summed in fp32 in a scrambled order.  The bound is taken at every vector's own R in turn: the tightest case
    there is.  -> by how much the two tests (all components, the first half of the steps) admit the vectors, and R."""
    f8 = np.float64
    n, d = y.shape
    subs, top, eta, square_loss = d // m, TOP[dtype], B["eta"], B["square_loss"]
    word_max = np.sqrt((y.reshape(n, subs, m).astype(f8) ** 2).sum(2).max()) * B["word_norm_slack"]
    part = np.concatenate([np.arange(0, d // 4), np.arange(d // 2, 3 * d // 4)])      # what the first half of the steps covers
    diff = (y - r).reshape(n, subs, m)
    ent = np.zeros((n, subs), np.float32)
    for t in range(m):
        ent = (diff[:, :, t].astype(f8) ** 2 + ent).astype(np.float32)
    R = np.zeros(n, np.float32)
    for j in range(subs):
        R = R + stored_entry(ent[:, j], dtype, truncate)
    rb, yb = bf16_round(r), bf16_round(y)
    n2 = (rb.reshape(subs, m).astype(f8) ** 2).sum(1)
    entry_max = (np.sqrt(n2 * B["rounded_norm"]) + word_max) ** 2 * B["entry_slack"]
    hidden = np.maximum(entry_max - top, 0).sum() * B["hidden_slack"] if np.isfinite(top) else 0.0
    wide = ((R * B["scale"] + B["add"] + hidden) * (1 + eta * B["limit_share"])).astype(np.float32)
    margins = []
    for cols, norm, less in ((np.arange(d), (r.astype(f8) ** 2).sum(), 0.0), (part, (rb[part].astype(f8) ** 2).sum(), square_loss)):
        start = (0.5 * (wide - (1 - eta - less) * norm)).astype(np.float32)
        need = (0.5 * (1 - eta - square_loss) * (yb[:, cols].astype(f8) ** 2).sum(1)).astype(np.float32)
        acc = start.copy()
        for t in rng.permutation(cols):
            acc = (acc + rb[t] * yb[:, t]).astype(np.float32)
        margins.append(acc - need)
    return margins, R


@pytest.mark.parametrize("dtype,truncate", [(0, False), (1, False), (2, False), (2, True), (3, False), (3, True)])
@pytest.mark.parametrize("d,m,scale", [(128, 2, 20.0), (96, 2, 0.05), (128, 4, 60.0), (64, 4, 1e-3)])
def test_filter_admits_every_survivor(library_bound, dtype, truncate, d, m, scale):
    # The library's constants.  Queries a little and far (6 sigma a component: half and e4m4 entries saturate at scale 60) off the cluster.
    rng = np.random.default_rng(d * 10 + m + dtype)
    B = library_bound(dtype, truncate, d // m, d)
    for far in (1.0, 6.0):
        r = (rng.standard_normal((12, d)) * scale * far).astype(np.float32)
        y = (rng.standard_normal((300, d)) * scale).astype(np.float32)
        y[:150] = (r[rng.integers(0, 12, 150)] + rng.standard_normal((150, d)) * scale * 0.3).astype(np.float32)
        for q in range(12):
            margins, R = filter_margins(r[q], y, dtype, truncate, m, B, rng)
            assert all(np.all(margin >= 0) for margin in margins)
            # the ball: no pair is left out whose cluster holds a vector with R <= bound
            radius = np.sqrt((y.astype(np.float64) ** 2).sum(1).max())
            gap = np.sqrt((r[q].astype(np.float64) ** 2).sum()) * B["cull_near"] - radius * B["cull_radius"]
            if R.min() < TOP[dtype] * B["cull_top"] and gap > 0:
                assert gap * gap <= (R.min() * B["scale"] + B["add"]) * B["cull_limit"]


@pytest.mark.parametrize("d,m", [(64, 4), (96, 2), (128, 2)])
def test_filter_bound_covers_the_worst_roundings_and_is_needed(library_bound, d, m):
    # Every component rounds to bf16 by the most there is, and the same way (257 -> 256).  A vector equal to the residual: its
    # product is short by twice 2^-8, which eta pays for.  Vectors straight opposite, with entries that saturate: what half
    # tables hide is reckoned from the rounded residual.  Numbers a little smaller than the library's would lose them.
    rng = np.random.default_rng(d)
    sign = np.where(rng.random(d) < 0.5, np.float32(-1), np.float32(1))
    r = (257 * sign).astype(np.float32)
    B = library_bound(0, False, d // m, d)
    ok = lambda y, dtype, numbers: all(np.all(v >= 0) for v in filter_margins(r, y, dtype, False, m, numbers, rng)[0])
    same = np.stack([r, r])
    assert ok(same, 0, B) and not ok(same, 0, dict(B, eta=0.25 * B["eta"], square_loss=0.0))
    H = library_bound(1, False, d // m, d)
    opposite = np.stack([-72 * sign, -72 * sign]).astype(np.float32)
    assert ok(opposite, 1, H) and not ok(opposite, 1, dict(H, rounded_norm=1.0))
    # a stored entry short by the whole share of its format: one-byte entries just under the middle of two codes
    for dtype, truncate in ((2, False), (2, True), (3, False), (3, True)):
        E = library_bound(dtype, truncate, d // m, d)
        f = np.float32(2.0 ** 10) * np.float32(1 + 2.0 ** -(3 if dtype == 2 else 4) * (0.999 if truncate else 0.4995))
        stored = stored_entry(np.array([f]), dtype, truncate)[0]
        assert stored < f and f <= stored * E["scale"]
        weaker = library_bound(dtype, False, d // m, d)["scale"] if truncate else 1 + 2.0 ** -15
        assert not f <= stored * weaker
