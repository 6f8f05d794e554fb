"""Timed workloads of the embedding-bag library, through its public entry points.

Three kinds of call make up the one-GPU work of a DLRM-style embedding layer:

  forward       pooled lookups (``EmbeddingBagTables.forward`` / ``forward_ex``): sum, mean or
                weighted sum of the rows each bag names, from fp32 / fp16 / bf16 tables, with int64
                or int32 ids, whole tables or one GPU's block of rows, with or without hit counts;
  bucketize     the send side of the row-wise exchange (``eb_bucketize_ex``): a mini-batch's ids
                sorted by the GPU whose row block holds them;
  sum_partials  its receive side (``sum_partials``): the partial results of every GPU added up.

``listed`` names fixed workloads, ``draw`` gives further ones from the same ranges.  Tables hold
N(0, 0.01); skewed ids follow a bounded power law over the ranks, spread over the table by a
permutation unless the case says that ranks are the ids.
"""
import math

import numpy as np
import torch

from paper_2512_05831_amd import eb

TORCH_DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
INDEX_DTYPES = {"i64": torch.int64, "i32": torch.int32}
INDEX_CODES = {"i64": eb.EB_IDX_I64, "i32": eb.EB_IDX_I32}

FORWARD = dict(op="forward", tables=1, rows=100_000, dim=64, dtype="f32", bags=256, len_lo=20, len_hi=20,
               p_empty=0.0, ids="uniform", alpha=0.0, permuted=True, index="i64", mode="sum", weights=False,
               hint=False, shards=1, hits=False)
BUCKETIZE = dict(op="bucketize", tables=8, rows=1_000_000, bags=256, len_lo=40, len_hi=40, p_empty=0.0,
                 ids="uniform", alpha=0.0, permuted=True, index="i64", destinations=8)
SUM_PARTIALS = dict(op="sum_partials", blocks=8, bags=2048, tables=8, dim=128, mean=False, len_lo=1, len_hi=100,
                    p_empty=0.02)


def listed():
    f = lambda name, **kw: dict(FORWARD, name=name, **kw)  # noqa: E731
    b = lambda name, **kw: dict(BUCKETIZE, name=name, **kw)  # noqa: E731
    return [
        # One sparse feature of one request batch: the smallest call, latency only.
        f("single_table_small", hint=True),
        # Online serving of many features at once, 128-byte rows, batch 128, pooling 16.
        f("many_tables_small_batch", tables=64, dim=32, bags=128, len_lo=16, len_hi=16, hint=True),
        # Ordinary inference batch, tables far larger than the caches, ids without reuse.
        f("uniform_f32", tables=8, rows=1_000_000, dim=128, bags=2048, len_lo=40, len_hi=40, hint=True),
        # The largest: an offline / training-size DLRM batch, 26 features, skewed ids, ragged bags.
        f("skewed_ragged_mean_f32", tables=26, rows=2_000_000, dim=128, bags=16384, len_lo=1, len_hi=100,
          p_empty=0.02, ids="zipf", alpha=1.05, mode="mean"),
        # Half-precision narrow rows with 32-bit ids: 64-byte rows, bound by accesses.
        f("narrow_bf16_i32", tables=16, rows=1_000_000, dim=32, dtype="bf16", bags=4096, len_lo=64, len_hi=64,
          index="i32", hint=True),
        # User-history features scored for one request batch: few, long, weighted bags.
        f("history_weighted_f16", tables=4, rows=1_000_000, dim=64, dtype="f16", bags=64, len_lo=200,
          len_hi=2000, ids="zipf", alpha=1.05, weights=True),
        # One GPU's row block of a 400M-id table under row-wise parallelism, with hit counts.
        f("row_shard_hits_f16", rows=400_000_000, dim=256, dtype="f16", bags=65536, len_lo=80, len_hi=80,
          ids="zipf", alpha=0.9, permuted=False, shards=8, hits=True),
        # A width from a rule of thumb on the row count, 6 * N^(1/4): odd rows of 378 bytes.
        f("odd_width_mean_f16_i32", tables=8, rows=1_000_000, dim=189, dtype="f16", bags=4096, len_lo=1,
          len_hi=50, p_empty=0.02, ids="zipf", alpha=1.05, index="i32", mode="mean"),
        # Exchange, send side: a small serving batch per GPU,
        b("bucketize_small"),
        # one GPU's mini-batch of the large batch split over 8 GPUs,
        b("bucketize_step_i32", tables=26, rows=2_000_000, bags=2048, len_lo=1, len_hi=100, p_empty=0.02,
          ids="zipf", alpha=1.05, index="i32"),
        # and the whole large batch.
        b("bucketize_batch", tables=26, rows=2_000_000, bags=16384, len_lo=1, len_hi=100, p_empty=0.02,
          ids="zipf", alpha=1.05),
        # Exchange, receive side, of that mini-batch: mean pooling finished after the sum.
        dict(SUM_PARTIALS, name="sum_partials_mean", tables=26, mean=True),
    ]


# ------------------------------------------------------------------------------- drawn cases


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lengths(rng, mean):
    """Fixed lengths, or uniform over a range around the same mean with a few empty bags."""
    if rng.random() < 0.4:
        return dict(len_lo=mean, len_hi=mean, p_empty=0.0)
    return dict(len_lo=1, len_hi=2 * mean - 1, p_empty=0.02)


def _ids(rng):
    if rng.random() < 0.5:
        return dict(ids="uniform", alpha=0.0)
    return dict(ids="zipf", alpha=round(rng.uniform(0.8, 1.2), 2))


def _mean_len(case):
    return (1.0 - case["p_empty"]) * (case["len_lo"] + case["len_hi"]) / 2.0


def draw(rng):
    kind = rng.choices(["forward", "history", "shard", "bucketize", "sum_partials"], [10, 2, 2, 5, 2])[0]
    index = rng.choice(["i64", "i32"])
    if kind == "bucketize":
        # 50,000 to 20 million ids, a bag every 1 to 100 of them.
        tables, ids = rng.randint(1, 40), _log_int(rng, 50_000, 20_000_000)
        mean = _log_int(rng, 1, 100)
        bags = max(1, min(ids // (tables * mean), 2_000_000 // tables))
        return dict(BUCKETIZE, tables=tables, rows=_log_int(rng, 10_000, 4_000_000), bags=bags, index=index,
                    destinations=rng.choice([2, 3, 4, 5, 8, 8, 8, 16, 32, 64]), **_lengths(rng, mean), **_ids(rng))
    if kind == "sum_partials":
        # 1 to 250 MB of partial results.
        blocks, tables, dim = rng.choice([2, 4, 8, 8, 16]), rng.randint(1, 64), rng.randint(4, 256)
        bags = max(1, _log_int(rng, 1_000_000, 250_000_000) // (4 * blocks * tables * dim))
        return dict(SUM_PARTIALS, blocks=blocks, tables=tables, dim=dim, bags=bags, mean=rng.random() < 0.5)
    dtype = rng.choice(["f32", "f16", "bf16"])
    mode = rng.choice(["sum", "sum", "mean"])
    dim = rng.choice([16, 32, 64, 64, 96, 128, 128, 256, 512]) if rng.random() < 0.6 else rng.randint(6, 300)
    row_bytes = dim * (4 if dtype == "f32" else 2)
    case = dict(FORWARD, dim=dim, dtype=dtype, index=index, mode=mode, weights=mode == "sum" and rng.random() < 0.25,
                hits=rng.random() < 0.25, **_ids(rng))
    if kind == "history":
        mean = _log_int(rng, 300, 3000)
        case.update(tables=rng.randint(1, 8), rows=_log_int(rng, 100_000, 2_000_000), bags=_log_int(rng, 4, 128),
                    len_lo=mean // 2, len_hi=mean + mean // 2)
    else:
        if kind == "shard":
            case.update(tables=rng.randint(1, 4), rows=_log_int(rng, 1_000_000, 50_000_000),
                        shards=rng.choice([2, 4, 8, 16]), bags=_log_int(rng, 1000, 65536), hits=rng.random() < 0.7)
        else:
            case.update(tables=_log_int(rng, 1, 64), rows=_log_int(rng, 10_000, 4_000_000),
                        bags=_log_int(rng, 64, 16384))
        case.update(_lengths(rng, _log_int(rng, 1, 100)))
        # No more row bytes than 4 GB, no more ids than 20 million.
        most = min(4e9 / row_bytes * case["shards"], 2e7)
        while case["tables"] * case["bags"] * _mean_len(case) > most:
            case["bags"] = max(1, case["bags"] * 2 // 3)
    while case["tables"] * (case["rows"] // case["shards"]) * row_bytes > 8e9:  # of table memory
        case["rows"] = case["rows"] * 2 // 3
    # Ids drawn without skew from tables beyond the caches: what the streaming hint is for.
    case["hint"] = case["ids"] == "uniform" and rng.random() < 0.8
    return case


# ------------------------------------------------------------------------------- inputs


def _generator(case, seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 16 + what)
    return g


def _offsets(case, seed):
    """Offsets of every (table, bag) as int64 on the GPU: lengths evenly spread over the case's
    range with its share of empty bags, in an order drawn from the seed."""
    n = case["tables"] * case["bags"]
    empty = int(round(case["p_empty"] * n))
    lo, span = case["len_lo"], case["len_hi"] + 1 - case["len_lo"]
    k = torch.arange(n - empty, device="cuda")
    lengths = torch.zeros(n, dtype=torch.int64, device="cuda")
    lengths[empty:] = lo + k * span // max(1, n - empty)
    lengths = lengths[torch.randperm(n, generator=_generator(case, seed, 1), device="cuda")]
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lengths, 0, out=off[1:])
    return off


def _indices(case, seed, off):
    """Row ids of every table's bags, one table after another (int64)."""
    rows, bags, g = case["rows"], case["bags"], _generator(case, seed, 2)
    ends = off[::bags].tolist()
    out = torch.empty(ends[-1], dtype=torch.int64, device="cuda")
    for t in range(case["tables"]):
        n = ends[t + 1] - ends[t]
        if case["ids"] == "uniform":
            ids = torch.randint(0, rows, (n,), generator=g, device="cuda")
        else:
            # Inverse of the continuous power law on [1, rows + 1), rounded down to a rank.
            q = 1.0 - case["alpha"]
            u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
            if abs(q) < 1e-9:
                x = torch.exp(u * math.log(rows + 1.0))
            else:
                x = (u * ((rows + 1.0) ** q - 1.0) + 1.0) ** (1.0 / q)
            ids = (x.to(torch.int64) - 1).clamp_(0, rows - 1)
            if case["permuted"]:
                ids = torch.randperm(rows, generator=g, device="cuda")[ids]
        out[ends[t]:ends[t + 1]] = ids
    return out


def _batch(case, seed):
    off = _offsets(case, seed)
    idx = _indices(case, seed, off)
    kind = INDEX_DTYPES[case["index"]]
    return off.to(kind), idx.to(kind)


def prepare(case, seed):
    if case["op"] == "forward":
        g = _generator(case, seed, 0)
        stored = case["rows"] // case["shards"]
        tables = [torch.empty((stored, case["dim"]), dtype=TORCH_DTYPES[case["dtype"]], device="cuda")
                  .normal_(0.0, 0.01, generator=g) for _ in range(case["tables"])]
        off, idx = _batch(case, seed)
        weights = None
        if case["weights"]:
            weights = torch.rand(idx.numel(), generator=_generator(case, seed, 3), device="cuda")
        handle = eb.EmbeddingBagTables(tables, rows=[case["rows"]] * case["tables"], shard_lo=0, shard_hi=stored) \
            if case["shards"] > 1 else eb.EmbeddingBagTables(tables)
        mode = (eb.EB_MEAN if case["mode"] == "mean" else eb.EB_SUM) | (eb.EB_HINT_STREAM_ROWS if case["hint"] else 0)
        plain = case["index"] == "i64" and weights is None
        return dict(op="forward", handle=handle, off=off, idx=idx, weights=weights, mode=mode, plain=plain,
                    bags=case["bags"], tables=case["tables"], hits=case["hits"])
    if case["op"] == "bucketize":
        T, B, G = case["tables"], case["bags"], case["destinations"]
        off, idx = _batch(case, seed)
        row = torch.tensor([g * case["rows"] // G for g in range(G + 1)], dtype=torch.int64)
        nbytes = eb.eb_bucketize_workspace(T, B, G)
        return dict(op="bucketize", T=T, B=B, G=G, off=off, idx=idx, bounds=row.repeat(T, 1).cuda(),
                    code=INDEX_CODES[case["index"]],
                    out_off=torch.empty((G, T * B + 1), dtype=torch.int64, device="cuda"),
                    out_idx=torch.empty_like(idx), seg=torch.empty(G + 1, dtype=torch.int64, device="cuda"),
                    ws=torch.empty(nbytes, dtype=torch.uint8, device="cuda"), nbytes=nbytes)
    G, B, T, D = case["blocks"], case["bags"], case["tables"], case["dim"]
    partials = torch.empty((G, B, T * D), dtype=torch.float32, device="cuda") \
        .normal_(0.0, 0.05, generator=_generator(case, seed, 0))
    off = _offsets(case, seed) if case["mean"] else None
    return dict(op="sum_partials", partials=partials, B=B, T=T, D=D, off=off,
                nnz=int(off[-1]) if case["mean"] else 0,
                out=torch.empty((B, T * D), dtype=torch.float32, device="cuda"))


# ------------------------------------------------------------------------------- one pass


def run(s):
    if s["op"] == "forward":
        if s["plain"]:
            return s["handle"].forward(s["idx"], s["off"], s["bags"], mode=s["mode"], hits=s["hits"])
        hits = torch.empty((s["bags"], s["tables"]), dtype=torch.int32, device="cuda") if s["hits"] else None
        return s["handle"].forward_ex(s["idx"], s["off"], s["bags"], mode=s["mode"], hits=hits, weights=s["weights"])
    if s["op"] == "bucketize":
        # A program that exchanges every batch keeps its send buffers and the workspace.
        eb.eb_bucketize_ex(s["T"], s["B"], s["G"], s["bounds"].data_ptr(), s["code"], s["idx"].data_ptr(),
                           s["idx"].numel(), s["off"].data_ptr(), s["out_off"].data_ptr(), s["out_idx"].data_ptr(),
                           s["out_idx"].numel(), s["seg"].data_ptr(), s["ws"].data_ptr(), s["nbytes"],
                           torch.cuda.current_stream().cuda_stream)
        return s["out_off"], s["out_idx"], s["seg"]
    return eb.sum_partials(s["partials"], s["B"], s["T"], s["D"], mean_offsets=s["off"], nnz=s["nnz"], out=s["out"])


# ------------------------------------------------------------------------------- what a pass needs


def _distinct_rows(case, n):
    """Expected number of distinct stored rows among n lookups of one table."""
    rows, stored = case["rows"], case["rows"] // case["shards"]
    if n <= 0:
        return 0.0
    if case["ids"] == "uniform":
        return stored * -math.expm1(n * math.log1p(-1.0 / rows)) if rows > 1 else 1.0
    # Ranks in runs that grow by under 1%, one probability for each run's ranks.
    edges = np.unique(np.concatenate([np.arange(1, 200), np.floor(np.geomspace(200, rows + 1, 4000)),
                                      [rows + 1.0]]))
    edges = edges[edges <= rows + 1]
    q = 1.0 - case["alpha"]
    cdf = np.log(edges) / math.log(rows + 1.0) if abs(q) < 1e-9 else (edges ** q - 1.0) / ((rows + 1.0) ** q - 1.0)
    p, count = np.diff(cdf) / np.diff(edges), np.diff(edges)
    if case["shards"] > 1 and not case["permuted"]:  # ranks are ids: only the first ones are stored
        count = np.clip(np.minimum(edges[1:], stored + 1) - np.minimum(edges[:-1], stored + 1), 0, None)
        return float(np.sum(count * -np.expm1(n * np.log1p(-np.minimum(p, 1 - 1e-12)))))
    return float(np.sum(count * -np.expm1(n * np.log1p(-np.minimum(p, 1 - 1e-12))))) / case["shards"]


def _local_share(case):
    """Share of the lookups that fall in the stored rows."""
    rows, stored = case["rows"], case["rows"] // case["shards"]
    if case["shards"] == 1 or case["permuted"] or case["ids"] == "uniform":
        return stored / rows
    q = 1.0 - case["alpha"]
    return math.log(stored + 1.0) / math.log(rows + 1.0) if abs(q) < 1e-9 \
        else ((stored + 1.0) ** q - 1.0) / ((rows + 1.0) ** q - 1.0)


def work(case):
    """Every distinct row, id, offset, weight and partial result read once, every result written once."""
    if case["op"] == "sum_partials":
        n = case["bags"] * case["tables"] * case["dim"]
        off = 8.0 * (case["bags"] * case["tables"] + 1) if case["mean"] else 0.0
        return {"bytes": 4.0 * n * (case["blocks"] + 1) + off, "flops": float(n * case["blocks"])}
    bags, ib = case["tables"] * case["bags"], 8 if case["index"] == "i64" else 4
    n = bags * _mean_len(case)
    if case["op"] == "bucketize":
        G = case["destinations"]
        return {"bytes": 2.0 * ib * n + ib * (bags + 1.0) + 8.0 * G * (bags + 1) + 8.0 * (case["tables"] + 1) * (G + 1),
                "flops": 0.0}
    row = case["dim"] * (4 if case["dtype"] == "f32" else 2)
    rows = case["tables"] * _distinct_rows(case, n / case["tables"])
    per_id = ib + (4 if case["weights"] else 0)
    per_bag = ib + 4 * case["dim"] + (4 if case["hits"] else 0)
    return {"bytes": rows * row + n * per_id + bags * per_bag,
            "flops": n * _local_share(case) * case["dim"] * (2.0 if case["weights"] else 1.0)}


def tolerance(case):
    # Ids, offsets and segments are whole numbers.  Pooled sums are 32-bit sums of the stored
    # values in some order, which measured up to 1.2e-7 off 64 bits for bags of up to 100 ids and
    # 4.9e-7 for bags of thousands.
    if case["op"] == "bucketize":
        return "exact"
    return {"rel": 2e-6, "max": 4e-5}


def exact(case, seed):
    """The same results in 64 bits, from plain tensor operations."""
    if case["op"] == "bucketize":
        return None
    s = prepare(case, seed)
    T, B = case["tables"], case["bags"]
    if case["op"] == "sum_partials":
        out = torch.zeros((B, T * case["dim"]), dtype=torch.float64, device="cuda")
        for block in s["partials"]:
            out += block
        if case["mean"]:
            lengths = (s["off"][1:] - s["off"][:-1]).view(T, B).t()[:, :, None]
            out = out.view(B, T, case["dim"]) / lengths.clamp(min=1) * (lengths > 0)  # an empty bag's mean is 0
            out = out.view(B, -1)
        return out
    off, idx, D = s["off"].to(torch.int64), s["idx"], case["dim"]
    lengths, ends = off[1:] - off[:-1], off[::B].tolist()
    out = torch.zeros((T, B, D), dtype=torch.float64, device="cuda")
    hits = torch.zeros((T, B), dtype=torch.int64, device="cuda")
    step = max(1, (1 << 27) // D)
    for t, table in enumerate(s["handle"].tables):
        bag = torch.repeat_interleave(torch.arange(B, device="cuda"), lengths[t * B:(t + 1) * B])
        for k in range(0, ends[t + 1] - ends[t], step):
            at = slice(ends[t] + k, min(ends[t] + k + step, ends[t + 1]))
            ids, to = idx[at].to(torch.int64), bag[k:k + step]
            ok = ids < table.shape[0]
            rows = table[ids.clamp(max=table.shape[0] - 1)].to(torch.float64) * ok[:, None]
            if s["weights"] is not None:
                rows *= s["weights"][at].to(torch.float64)[:, None]
            out[t].index_add_(0, to, rows)
            hits[t].index_add_(0, to, ok.to(torch.int64))
    if case["mode"] == "mean":
        out /= lengths.view(T, B, 1).clamp(min=1)
    out = out.permute(1, 0, 2).reshape(B, T * D)
    return (out, hits.t().to(torch.int32).contiguous()) if case["hits"] else out
