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


@pytest.mark.parametrize("dtype,truncate", [(0, False), (1, False), (2, False), (2, True), (3, False), (3, True)])
@pytest.mark.parametrize("d,m,scale", [(128, 2, 20.0), (96, 2, 0.05), (128, 4, 60.0), (64, 4, 1e-3)])
def test_filter_admits_every_survivor(dtype, truncate, d, m, scale):
    # The host's constants and the kernel's arithmetic, emulated: residuals and codewords in bf16, the product and its start
    # summed in fp32 in a scrambled order.  The bound is taken at every vector's own R in turn: the tightest case there is.
    # Queries a little and far (6 sigma a component: half and e4m4 entries saturate at scale 60) off the cluster.
    rng = np.random.default_rng(d * 10 + m + dtype)
    f8 = np.float64
    for far in (1.0, 6.0):
        r = (rng.standard_normal((12, d)) * scale * far).astype(np.float32)
        y = (rng.standard_normal((300, d)) * scale).astype(np.float32)
        y[:150] = (r[rng.integers(0, 12, 150)] + rng.standard_normal((150, d)) * scale * 0.3).astype(np.float32)
        loss = {0: 0.0, 1: 1 / 2048, 2: 1 / (9 if truncate else 17), 3: 1 / (17 if truncate else 33)}[dtype]
        top = {0: np.inf, 1: 65504.0, 2: 122880.0, 3: 1.9375 * 2.0 ** 14}[dtype]
        subs = d // m
        grow = (1 + 2.0 ** -15) / (1 - loss)
        add = (subs * 2.0 ** -25 if dtype == 1 else 0.0) / (1 - loss) * 1.001 + 1e-30
        eta = 0.00392 + (12 * d + 64) * 2.0 ** -24
        word_max = np.sqrt((y.reshape(300, subs, m).astype(f8) ** 2).sum(2).max()) * 1.0001
        part = np.concatenate([np.arange(0, d // 4), np.arange(d // 2, 3 * d // 4)])      # what the first half of the steps covers
        for q in range(12):
            diff = (y - r[q]).reshape(300, subs, m)
            ent = np.zeros((300, subs), np.float32)
            for t in range(m):
                ent = (diff[:, :, t].astype(f8) ** 2 + ent).astype(np.float32)
            R = np.zeros(300, np.float32)
            for j in range(subs):
                R = R + stored_entry(ent[:, j], dtype, truncate)
            rb, yb = bf16_round(r[q]), bf16_round(y)
            n2 = (rb.reshape(subs, m).astype(f8) ** 2).sum(1)
            hidden = np.maximum((np.sqrt(n2 * 1.008) + word_max) ** 2 * 1.00001 - top, 0).sum() * 1.0001 if np.isfinite(top) else 0.0
            wide = ((R * grow + add + hidden) * (1 + eta / 16)).astype(np.float32)
            rr = (r[q].astype(f8) ** 2).sum()
            for cols, norm, less in ((np.arange(d), rr, 0.0), (part, (rb[part].astype(f8) ** 2).sum(), 0.00394)):
                start = (0.5 * (wide - (1 - eta - less) * norm)).astype(np.float32)
                need = (0.5 * (1 - eta - 0.00394) * (yb[:, cols].astype(f8) ** 2).sum(1)).astype(np.float32)
                acc = start.copy()
                for t in rng.permutation(cols):
                    acc = (acc + rb[t] * yb[:, t]).astype(np.float32)
                assert np.all(acc >= need)
            # the ball: no pair is left out whose cluster holds a vector with R <= bound
            radius = np.sqrt((y.astype(f8) ** 2).sum(1).max())
            gap = np.sqrt(rr) * 0.99987 - radius * 1.00013
            least = R.min()
            if least < top * 0.9999 and gap > 0:
                assert gap * gap <= (least * grow + add) * 1.0001
