"""The work that users of this library have it do, as cases that can be timed and compared.

A case is one call (or one short sequence of calls) through the Python binding on inputs of a stated size.  The
vectors are the two synthetic families the repository is measured on, drawn on the GPU: "grid", 128-d integer-valued
descriptors (1,000 Gaussian components, sigma 20, clipped to 0..255), and "unit", 96-d unit-norm descriptors (2,000
components, sigma 0.05).  Queries come from the same mixture as the indexed vectors.

  op         what one pass does
  search     Index.ivfpq_search: probe selection, lookup tables, code scan, top-k
  rerank     a search for `wide` candidates, then ivfpq_refine down to k with the stored vectors
  assign     ivfpq_assign_device: the nearest of many centres for every row (k-means assignment, inserting new rows)
  build      Index.ivfpq_build_device and ivfpq_index_export: an index made and saved
  open       Index.ivfpq_index_from_arrays and ivfpq_upload of a saved index, then its first batch of queries
"""
import math

import torch

import paper_2301_06672_amd as ivfpq

DIM = {"grid": 128, "unit": 96}
TABLES = {"fp32": ivfpq.LUT_FP32, "fp16": ivfpq.LUT_FP16, "e5m3": ivfpq.LUT_FP8_E5M3, "e4m4": ivfpq.LUT_FP8_E4M4}
E4M4_BIAS = {"grid": 1, "unit": 16}      # puts the format's 16 binades on the entries of each family
BUILD_ITERS = 6                          # Lloyd iterations of a measured build
INDEX_ITERS = 4                          # ... and of the indexes that the other cases only hold


def _search(name, data, n, lists, sub, bits, nq, probes, k, table):
    return {"name": name, "op": "search", "data": data, "n": n, "lists": lists, "sub": sub, "bits": bits, "nq": nq,
            "probes": probes, "k": k, "table": table}


def listed():
    return [
        # an interactive service: one query at a time on 10^6 vectors, where launches and latency count
        _search("one query", "grid", 1_000_000, 1024, 64, 8, 1, 20, 10, "e5m3"),
        # a server's micro-batch of the unit-norm set, half-precision tables
        _search("64 queries", "unit", 1_000_000, 1024, 48, 8, 64, 20, 10, "fp16"),
        # an odd, middling batch with full-precision tables and short codes
        _search("777 queries float table", "grid", 1_000_000, 1024, 32, 8, 777, 33, 50, "fp32"),
        # offline batch search on 10^6 vectors, the configuration of the repository's smaller benchmark
        _search("batch on 1M", "grid", 1_000_000, 1024, 64, 8, 10_000, 20, 10, "e5m3"),
        # the 10^7 unit-norm set at the paper's k
        _search("batch on 10M", "unit", 10_000_000, 10_000, 48, 8, 10_000, 50, 100, "e5m3"),
        # lists of 2,000 vectors, 32-byte codes, 64 probes, k = 100: the shape of the 10^8-vector benchmark at a
        # size that can be built in seconds
        _search("batch long lists", "grid", 10_000_000, 5_000, 32, 8, 10_000, 64, 100, "e5m3"),
        # the same with 4-bit codes and half tables
        _search("batch 4-bit codes", "grid", 4_000_000, 2_000, 64, 4, 10_000, 64, 100, "fp16"),
        # bit-packed codes
        _search("batch 7-bit codes", "grid", 1_000_000, 1024, 64, 7, 10_000, 20, 10, "e5m3"),
        # high-recall search: 40 candidates re-ranked to 10 with the stored vectors
        {"name": "search and re-rank", "op": "rerank", "data": "grid", "n": 1_000_000, "lists": 1024, "sub": 64, "bits": 8,
         "nq": 4_096, "probes": 20, "wide": 40, "k": 10, "table": "e5m3"},
        # new rows given to the clusters of an existing index
        {"name": "assign rows", "op": "assign", "data": "unit", "n": 500_000, "lists": 10_000},
        # index construction
        {"name": "build on 1M", "op": "build", "data": "grid", "n": 1_000_000, "lists": 1024, "sub": 64, "bits": 8},
        # a server that starts: a saved index opened, and its first queries
        {"name": "open and search", "op": "open", "data": "unit", "n": 1_000_000, "lists": 1024, "sub": 48, "bits": 8,
         "nq": 256, "probes": 20, "k": 10, "table": "e5m3"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["search", "rerank", "assign", "build", "open"], [8, 1, 1, 1, 1])[0]
    data = rng.choice(["grid", "unit"])
    if op == "assign":
        return {"op": op, "data": data, "n": _log_int(rng, 3_000, 500_000), "lists": _log_int(rng, 64, 9_000)}
    n = _log_int(rng, 20_000, 2_000_000 if op == "search" else 800_000)
    lists = max(32, int(n / rng.uniform(700, 2_500)))
    sub, bits = rng.choice([(64, 8), (32, 8), (64, 4), (64, 7), (64, 6)]) if data == "grid" else (48, rng.choice([8, 8, 4]))
    case = {"op": op, "data": data, "n": n, "lists": lists, "sub": sub, "bits": bits}
    if op == "build":
        return case
    case["nq"] = _log_int(rng, 1, 10_000 if op == "search" else 3_000)
    case["probes"] = min(lists, _log_int(rng, 1, 64))
    case["k"] = _log_int(rng, 1, 100)
    if op == "rerank":
        case["wide"] = min(1_000, case["k"] * rng.randint(2, 6))
    case["table"] = rng.choice(["fp32", "fp16", "e5m3", "e5m3", "e4m4"])
    return case


def _centres(data, gen):
    if data == "grid":
        return torch.rand((1_000, 128), generator=gen, device="cuda") * 128.0
    c = torch.randn((2_000, 96), generator=gen, device="cuda")
    return c / c.norm(dim=1, keepdim=True)


def _rows(data, centres, n, gen, chunk=1 << 20):
    out = torch.empty((n, DIM[data]), dtype=torch.float32, device="cuda")
    for at in range(0, n, chunk):
        rows = out[at:at + chunk]
        which = torch.randint(centres.shape[0], (rows.shape[0],), generator=gen, device="cuda")
        rows.normal_(generator=gen)
        rows.mul_(20.0 if data == "grid" else 0.05).add_(centres[which])
        if data == "grid":
            rows.clamp_(0.0, 255.0).round_()
        else:
            rows.div_(rows.norm(dim=1, keepdim=True))
    return out


def prepare(case, seed):
    """The program's own data: vectors, queries, and (but where that is what is measured) the built and uploaded index."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    op, data = case["op"], case["data"]
    centres = _centres(data, gen)
    rows = _rows(data, centres, case["n"], gen)
    state = {"case": case}
    if op == "assign":
        pick = torch.randperm(case["n"], generator=gen, device="cuda")[:case["lists"]]
        more = case["lists"] - pick.numel()
        start = rows[pick] if more <= 0 else torch.cat([rows[pick], _rows(data, centres, more, gen)])
        state.update(rows=rows, centres=start.contiguous())
        return state
    if op == "build":
        state.update(rows=rows, seed=int(seed))
        return state
    state["queries"] = _rows(data, centres, case["nq"], gen)
    index = ivfpq.Index.ivfpq_build_device(rows, case["lists"], case["sub"], case["bits"], INDEX_ITERS, seed=int(seed))
    if op == "open":
        state["saved"] = index.ivfpq_index_export()
        return state
    index.ivfpq_set_e4m4_bias(E4M4_BIAS[data])
    state["index"] = index.ivfpq_upload()
    if op == "rerank":
        state["rows"] = rows
    return state


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "assign":
        return ivfpq.ivfpq_assign_device(state["rows"], state["centres"])
    if op == "build":
        index = ivfpq.Index.ivfpq_build_device(state["rows"], case["lists"], case["sub"], case["bits"], BUILD_ITERS, seed=state["seed"])
        return index.ivfpq_index_export()
    if op == "open":
        index = ivfpq.Index.ivfpq_index_from_arrays(DIM[case["data"]], case["lists"], case["sub"], case["bits"], *state["saved"])
        index.ivfpq_set_e4m4_bias(E4M4_BIAS[case["data"]])
        return index.ivfpq_upload().ivfpq_search(state["queries"], case["probes"], case["k"], TABLES[case["table"]])
    index, queries, table = state["index"], state["queries"], TABLES[case["table"]]
    if op == "rerank":
        ids, _ = index.ivfpq_search(queries, case["probes"], case["wide"], table)
        return ivfpq.ivfpq_refine(state["rows"], queries, ids, case["k"])
    return index.ivfpq_search(queries, case["probes"], case["k"], table)


def work(case):
    """Every input read once, every output written once; multiply-adds as two operations, one addition per (scanned
    vector, sub-space) with lists of average length."""
    n, lists, d = case["n"], case["lists"], DIM[case["data"]]
    op = case["op"]
    if op == "assign":
        return {"bytes": 4 * d * (n + lists) + 4 * n, "flops": 2.0 * n * lists * d}
    code = case["sub"] * case["bits"] // 8
    book = case["sub"] << case["bits"]                      # codebook entries, d / sub components each
    index_bytes = 4 * lists * d + 4 * book * d // case["sub"] + n * (code + 8)
    if op == "build":
        train = min(n, 256 * lists)
        coarse = 2.0 * d * lists * (BUILD_ITERS * train + n)
        codes = 3.0 * d * (1 << case["bits"]) * (BUILD_ITERS * min(n, 262_144) + n)
        return {"bytes": 4 * d * n + index_bytes, "flops": coarse + codes}
    nq, probes, k = case["nq"], case["probes"], case["k"]
    met = 1.0 - (1.0 - probes / lists) ** nq                # share of the lists that some query probes
    flops = 2.0 * nq * lists * d + float(nq) * probes * (n / lists) * case["sub"]
    moved = 4 * d * (nq + lists) + 4 * book * d // case["sub"] + met * n * code + 12 * nq * k
    if op == "rerank":
        moved += 4 * d * min(n, nq * case["wide"])
        flops += 3.0 * nq * case["wide"] * d
    if op == "open":
        moved += 2 * index_bytes
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    """Index construction and assignment are decided by float64 distances: the same bits.  Distances are fp32 sums of
    up to 64 non-negative terms, and results that are closer than two orders of summation may change places: summed
    from the last sub-space instead of the first, the k = 100 best of both families differed by 3.0e-7 (norms),
    9.3e-7 (largest) and in 1e-4 of the ids.  Stated: four times that, and ten times for the ids, which grow closer
    with the size of the index."""
    if case["op"] in ("assign", "build"):
        return "exact"
    return {"rel": 1.2e-6, "max": 4e-6, "differ": 1e-3}
