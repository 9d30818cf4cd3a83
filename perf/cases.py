"""The calls that a user of the library makes, as cases to be timed and compared.

A case is one public call over a seeded table: rows are compressed and opened once, as a
program does at start-up, and one pass is one gather, one decompress, one cached gather or
one compress. The tables imitate the shapes and value structure of the benchmark's
workloads (GNN features, DLRM embedding tables, a bf16 KV cache, a sparse feature table)
and of the tests' wide rows; they are drawn on the GPU and are smaller than the largest
tables of the benchmark, so that a case is quick to prepare.

    listed()            the cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) the open handle, ids and output buffer of a program
    run(state)          one pass
    exact(case, seed)   the rows the pass has to return, from the generator itself
"""
import math

import numpy as np
import torch

import paper_2605_30728_amd as ibp

DEVICE = "cuda"
PLACEMENTS = {"device": ibp.IBP_OPEN_PAYLOAD_DEVICE, "staged": ibp.IBP_OPEN_PAYLOAD_HOST,
              "zero_copy": ibp.IBP_OPEN_PAYLOAD_HOST_ZERO_COPY}
TABLES = 26                # embedding tables of the DLRM lookups
ZIPF_S = 1.05              # popularity of their rows
HEAD_TOKENS = 32768        # rows of the KV cache that share a head (and its outlier channels)

# The share of a row's raw bytes that its packed form keeps, per kind of values, under
# per-cluster Masks and under one global Mask (T = 0.8 n, 8-byte chunks).
KEPT = {"gnn": (0.50, 0.54), "dlrm": (0.38, 0.70), "kv": (0.71, 0.86), "sparse": (0.51, 0.60)}


def listed():
    return [
        # one recommendation request: 8 candidates x 26 tables, ids arriving on the host
        # (latency and launches count)
        {"name": "lookup_small", "call": "gather_host_ids", "values": "dlrm", "rows": TABLES * 4000, "elems": 128,
         "group_rows": 32, "ids": "zipf", "n": 8 * TABLES},
        # a DLRM training batch: 2,048 samples x 26 Zipf lookups in [sample][table] order
        {"name": "dlrm_batch", "call": "gather", "values": "dlrm", "rows": TABLES * 40000, "elems": 128,
         "group_rows": 32, "ids": "zipf", "n": 2048 * TABLES},
        # a 2-hop GNN minibatch over an OGB-Products-like table: sorted unique ids, 400-byte rows
        {"name": "gnn_minibatch", "call": "gather", "values": "gnn", "rows": 2400000, "elems": 100,
         "group_rows": 32, "ids": "sorted", "n": 163840},
        # half an epoch of shuffled feature rows from a large sparse table
        {"name": "epoch_gather", "call": "gather", "values": "sparse", "rows": 3000000, "elems": 128,
         "group_rows": 64, "ids": "shuffled", "n": 1500000},
        # random rows of 4 KB (hidden states, wide embeddings): several tiles per row
        {"name": "wide_gather", "call": "gather", "values": "gnn", "rows": 100000, "elems": 1024,
         "group_rows": 32, "ids": "shuffled", "n": 16384},
        # one layer of a bf16 KV cache, K and V x 8 heads x 32,768 tokens x 128
        {"name": "kv_layer", "call": "decompress", "values": "kv", "rows": 524288, "elems": 128, "group_rows": 32},
        # a bf16 tensor whose rows are not a power of two (2,400 B, 600 words) and whose last
        # cluster is short, from inside a cluster to its end
        {"name": "wide_decompress", "call": "decompress", "values": "kv", "rows": 50021, "elems": 1200,
         "group_rows": 32, "first": 5},
        # the paper's own scheme (one global Mask, participation bits): the KV layer ...
        {"name": "kv_thresholded", "call": "decompress", "values": "kv", "rows": 524288, "elems": 128,
         "group_rows": 524288, "chunk_bytes": 8, "threshold_percent": 80},
        # ... and the GNN minibatch
        {"name": "gnn_thresholded", "call": "gather", "values": "gnn", "rows": 1200000, "elems": 100,
         "group_rows": 1200000, "chunk_bytes": 8, "threshold_percent": 80, "ids": "sorted", "n": 81920},
        # features larger than the GPU: host packing, PCIe and decode overlapped
        {"name": "gnn_staged", "call": "gather_host_ids", "values": "gnn", "rows": 1000000, "elems": 100,
         "group_rows": 32, "ids": "sorted", "n": 81920, "placement": "staged"},
        # embedding tables in host memory behind a compressed device cache of the popular rows
        {"name": "dlrm_cache", "call": "cache_gather", "values": "dlrm", "rows": TABLES * 20000, "elems": 128,
         "group_rows": 32, "ids": "zipf", "n": 2048 * TABLES, "placement": "zero_copy", "cached_percent": 12},
        # start-up: a table compressed on the host (the microbenchmark's tensors, half of whose
        # bits are the same in every row: a stream's size then does not depend on the seed)
        {"name": "compress_table", "call": "compress", "values": "fixed_bits", "fixed_percent": 50, "rows": 240000,
         "elems": 100, "group_rows": 32},
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    family = rng.choice(["lookup", "dlrm", "gnn", "epoch", "wide", "kv", "wide_rows", "kv_thresholded",
                         "gnn_thresholded", "host", "cache", "compress"])
    group = rng.choice([16, 24, 32, 64])
    if family in ("lookup", "dlrm"):
        small = family == "lookup"
        samples = _log(rng, 1, 64) if small else _log(rng, 32, 2048)
        return {"call": "gather_host_ids" if small or rng.random() < 0.3 else "gather", "values": "dlrm",
                "rows": TABLES * _log(rng, 2000, 4000 if small else 40000), "elems": _log(rng, 16, 128),
                "group_rows": group, "ids": "zipf", "n": samples * TABLES}
    if family == "gnn":
        rows = _log(rng, 50000, 1500000)
        return {"call": "gather", "values": rng.choice(["gnn", "sparse"]), "rows": rows, "elems": _log(rng, 32, 160),
                "group_rows": group, "ids": "sorted", "n": _log(rng, 1000, rows // 8)}
    if family == "epoch":
        rows = _log(rng, 400000, 2000000)
        return {"call": "gather", "values": rng.choice(["gnn", "sparse"]), "rows": rows, "elems": _log(rng, 64, 128),
                "group_rows": group, "ids": "shuffled", "n": rng.randint(rows // 8, rows // 2)}
    if family == "wide":
        rows = _log(rng, 5000, 100000)
        return {"call": "gather", "values": rng.choice(["gnn", "sparse", "dlrm"]), "rows": rows,
                "elems": rng.choice([_log(rng, 160, 512), _log(rng, 513, 1024)]), "group_rows": group,
                "ids": rng.choice(["sorted", "shuffled"]), "n": _log(rng, 500, min(rows, 16384))}
    if family == "kv":
        rows = _log(rng, 2048, 524288)
        first = rng.choice([0, rng.randint(0, rows // 2)])
        return {"call": "decompress", "values": rng.choice(["kv", "dlrm"]), "rows": rows, "elems": 2 * _log(rng, 16, 64),
                "group_rows": group, "first": first}
    if family == "wide_rows":
        rows = _log(rng, 500, 50000)
        first = rng.choice([0, rng.randint(0, rows // 2)])
        return {"call": "decompress", "values": rng.choice(["kv", "gnn"]), "rows": rows,
                "elems": 2 * rng.choice([_log(rng, 130, 512), _log(rng, 513, 600)]), "group_rows": group, "first": first}
    if family == "kv_thresholded":
        rows = _log(rng, 2048, 524288)
        return {"call": "decompress", "values": "kv", "rows": rows, "elems": 4 * _log(rng, 8, 32), "group_rows": rows,
                "chunk_bytes": rng.choice([4, 8]), "threshold_percent": rng.choice([80, 90])}
    if family == "gnn_thresholded":
        rows = _log(rng, 50000, 1200000)
        return {"call": "gather", "values": "gnn", "rows": rows, "elems": 2 * _log(rng, 16, 64), "group_rows": rows,
                "chunk_bytes": rng.choice([4, 8]), "threshold_percent": rng.choice([80, 90]), "ids": "sorted",
                "n": _log(rng, 1000, rows // 8)}
    if family == "host":
        rows = _log(rng, 50000, 800000)
        return {"call": "gather_host_ids", "values": rng.choice(["gnn", "sparse"]), "rows": rows,
                "elems": _log(rng, 32, 128), "group_rows": group, "ids": "sorted", "n": _log(rng, 1000, rows // 12),
                "placement": rng.choice(["staged", "zero_copy"])}
    if family == "cache":
        return {"call": "cache_gather", "values": "dlrm", "rows": TABLES * _log(rng, 4000, 20000),
                "elems": _log(rng, 16, 128), "group_rows": group, "ids": "zipf", "n": _log(rng, 32, 2048) * TABLES,
                "placement": "zero_copy", "cached_percent": rng.randint(8, 25)}
    return {"call": "compress", "values": "fixed_bits", "fixed_percent": rng.randint(10, 90),
            "rows": _log(rng, 10000, 240000), "elems": _log(rng, 32, 100), "group_rows": rng.choice([32, 48, 64])}


# ---------------------------------------------------------------- inputs

def _rng(seed, purpose):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 8 + purpose)
    return g


def _is_bf16(case):
    return case["values"] == "kv"


def _row_bytes(case):
    return case["elems"] * (2 if _is_bf16(case) else 4)


def _row_values(case, seed):
    """The table's rows on the GPU, float32 (bfloat16 for the KV cache)."""
    g = _rng(seed, 0)
    n, e = case["rows"], case["elems"]
    if case["values"] == "gnn":          # N(0, 1) rounded to 8 mantissa bits, ties to even
        u = torch.randn(n, e, generator=g, device=DEVICE).view(torch.int32)
        u += ((u >> 15) & 1) + 0x3FFF
        u &= -(1 << 15)
        return u.view(torch.float32)
    if case["values"] == "dlrm":         # U(-0.05, 0.05) in steps of 1/4096
        u = torch.rand(n, e, generator=g, device=DEVICE)
        return u.sub_(0.5).mul_(0.1 * 4096).round_().div_(4096)
    if case["values"] == "sparse":       # 70% zeros, the rest U(0, 1) in steps of 1/1024
        u = torch.rand(n, e, generator=g, device=DEVICE).mul_(1024).round_().div_(1024)
        return u.mul_(torch.rand(n, e, generator=g, device=DEVICE) >= 0.7)
    if case["values"] == "fixed_bits":   # that share of a row's bits is the same in every row, the rest uniform
        bits = e * 32
        fixed = torch.zeros(bits, dtype=torch.int64, device=DEVICE)
        fixed[torch.randperm(bits, generator=g, device=DEVICE)[:bits * case["fixed_percent"] // 100]] = 1
        keep = (fixed.view(e, 32) << torch.arange(32, device=DEVICE)).sum(1)
        word = lambda *shape: torch.randint(0, 1 << 32, shape, generator=g, device=DEVICE)  # noqa: E731
        keep, value = keep.to(torch.int32), word(e).to(torch.int32)
        return ((word(n, e).to(torch.int32) & ~keep) | (value & keep)).view(torch.float32)
    # 0.5 N(0, 1), two outlier channels x 20 in every head, rounded to bfloat16
    x = torch.randn(n, e, generator=g, device=DEVICE).mul_(0.5)
    heads = -(-n // HEAD_TOKENS)
    channel = torch.rand(heads, e, generator=g, device=DEVICE).argsort(1)[:, :2]
    for h in range(heads):
        x[h * HEAD_TOKENS:(h + 1) * HEAD_TOKENS, channel[h]] *= 20.0
    return x.to(torch.bfloat16)


def _popular(case, seed):
    """Per table, its rows in order of popularity."""
    per = case["rows"] // TABLES
    return torch.rand(TABLES, per, generator=_rng(seed, 1), device=DEVICE).argsort(1)


def _row_ids(case, seed):
    g, n, rows = _rng(seed, 2), case["n"], case["rows"]
    if case["ids"] == "sorted":
        return torch.randperm(rows, generator=g, device=DEVICE)[:n].sort()[0]
    if case["ids"] == "shuffled":
        return torch.randperm(rows, generator=g, device=DEVICE)[:n].contiguous()
    per = rows // TABLES                 # bounded Zipf ranks by inverse CDF
    w = torch.arange(1, per + 1, device=DEVICE, dtype=torch.float64) ** -ZIPF_S
    c = torch.cumsum(w, 0)
    u = torch.rand(n // TABLES, TABLES, generator=g, device=DEVICE, dtype=torch.float64) * c[-1]
    rank = torch.searchsorted(c, u).clamp_(max=per - 1)
    row = _popular(case, seed).gather(1, rank.t().contiguous()).t()
    return (row + torch.arange(TABLES, device=DEVICE) * per).reshape(-1).contiguous()


def _host_rows(case, seed):
    rows = _row_values(case, seed)
    return rows.view(torch.int16 if _is_bf16(case) else torch.int32).cpu().numpy()


# ---------------------------------------------------------------- the pass

class State:
    """What a program keeps between calls; it closes the handle when it goes."""

    def __init__(self):
        self.call = None
        self.handle = self.cache = self.ids = self.out = self.rows = None
        self.first = self.n = self.group_rows = 0

    def __del__(self):
        if self.cache is not None:
            ibp.ibp_cache_destroy(self.cache)
        if self.handle is not None:
            ibp.ibp_close(self.handle)


def _range(case):
    first = case.get("first", 0)
    return first, case["rows"] - first


def prepare(case, seed):
    s = State()
    s.call = case["call"]
    s.group_rows = case["group_rows"]
    rows = _host_rows(case, seed)
    if s.call == "compress":
        s.rows = rows
        return s
    if case.get("chunk_bytes"):
        stream = ibp.ibp_compress_ex(rows, s.group_rows, case["chunk_bytes"], (case["threshold_percent"], 100))
    else:
        stream = ibp.ibp_compress(rows, s.group_rows)
    s.handle = ibp.ibp_open(stream, torch.cuda.current_device(), PLACEMENTS[case.get("placement", "device")])
    if s.call == "decompress":
        s.first, s.n = _range(case)
    else:
        s.n = case["n"]
        s.ids = _row_ids(case, seed)
        if s.call == "gather_host_ids":
            s.ids = s.ids.cpu().numpy()
        if s.call == "cache_gather":
            per = case["rows"] // TABLES
            hot = _popular(case, seed)[:, :per * case["cached_percent"] // 100]
            hot = hot + torch.arange(TABLES, device=DEVICE)[:, None] * per
            s.cache = ibp.ibp_cache_create(s.handle, hot.t().reshape(-1).cpu().numpy())
    s.out = torch.empty(s.n, case["elems"], dtype=torch.bfloat16 if _is_bf16(case) else torch.float32, device=DEVICE)
    return s


def run(s):
    if s.call == "gather":
        ibp.ibp_gather_decompress_device(s.handle, s.ids, s.out)
    elif s.call == "gather_host_ids":
        ibp.ibp_gather_decompress(s.handle, s.ids, s.out)
    elif s.call == "decompress":
        ibp.ibp_decompress(s.handle, s.first, s.n, s.out)
    elif s.call == "cache_gather":
        ibp.ibp_cache_gather(s.cache, s.ids, s.out)
    else:
        return ibp.ibp_compress(s.rows, s.group_rows)
    return s.out


# ---------------------------------------------------------------- what a pass is compared with

def work(case):
    """Bytes read and written once: the ids, the packed rows, the rows themselves, and per
    cluster touched its offset and the distinct Mask/Bitval words with a 4-bit index per
    word (under one Mask: per row an offset). Nothing here computes on floats."""
    L, G = _row_bytes(case), case["group_rows"]
    if case["call"] == "compress":
        kept = 1 - case["fixed_percent"] / 100
        return {"bytes": case["rows"] * L * (1 + kept) + case["rows"] / G * 2 * L, "flops": 0}
    kept = KEPT[case["values"]][1 if case.get("chunk_bytes") else 0]
    n = _range(case)[1] if case["call"] == "decompress" else case["n"]
    clusters = -(-case["rows"] // G)
    touched = clusters if case["call"] == "decompress" else clusters * -math.expm1(-n / clusters)
    per_row = (0 if case["call"] == "decompress" else 8) + (8 if case.get("chunk_bytes") else 0)
    return {"bytes": n * (per_row + kept * L + L) + touched * (8 + 64 + L / 8), "flops": 0}


def tolerance(case):
    """The scheme is lossless: every bit of a row and of a stream is determined."""
    return "exact"


def exact(case, seed):
    if case["call"] == "compress":
        return None                      # a stream of bytes
    rows = _row_values(case, seed)
    if case["call"] == "decompress":
        first, n = _range(case)
        return rows[first:first + n].double()
    return rows[_row_ids(case, seed)].double()
