"""The lookups whose speed is measured: what a DLRM inference service has the library do.

A case names the tables (how many, how large, E, dtype), the queries (batch, lookups per
bag, skew) and the options (mean pooling, per-lookup weights).  ``prepare`` is what such a
service holds before a request: the tables on the device, a plan made from the statistics
of earlier queries and bound to the tables, one batch of device indices and offsets, and
the output buffer.  ``run`` is one ``Plan.lookup`` over that batch.

Sizes come from the repository's five workloads (``workloads/``) and from the shapes that
its random-configuration tests draw (row widths of 16 bytes to 1 KB, empty bags, long bags,
batches below the plan's largest).  Table bytes are capped at 24 GB so that several sets
of inputs fit the card.

Keys of a case:
  tables, rows_lo, rows_hi   tables of rows spaced geometrically from rows_lo to rows_hi
  big_rows, big_pf, big_alpha   one more table in front (0 rows: none), big_pf lookups per bag
  E, dtype                   row width and element type ("f32" | "f16")
  max_batch, batch           the plan's largest batch and this call's
  pf, pf_lo, pf_hi           lookups per bag: Poisson(pf) clipped to [pf_lo, pf_hi]; pf_lo =
                             pf_hi: exactly that many
  alpha                      Zipf exponent over a table's rows (0: uniform)
  mean, weighted             mean pooling of every table; an fp32 weight per lookup
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

import paper_2507_01676_amd as embx

TABLE_BYTES_CAP = 24e9
HISTORY_LOOKUPS = 16384   # lookups per table the planner's statistics come from
HOT_LISTED = 1024
VALUE = 0.05              # tables hold uniform values in [-VALUE, VALUE)


def _case(name, **kw):
    c = {"name": name, "big_rows": 0, "big_pf": 0, "big_alpha": 0.0, "mean": False, "weighted": False}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one small request over four small tables (workload 1)
        _case("online_e32", tables=4, rows_lo=100, rows_hi=100000, E=32, dtype="f32", max_batch=128, batch=128,
              pf=1.0, pf_lo=1, pf_hi=1, alpha=0.0),
        # a handful of queries with multi-hot features under a latency target: the batch is far
        # below the plan's largest
        _case("online_multihot_e64", tables=26, rows_lo=10, rows_hi=4000000, E=64, dtype="f32", max_batch=64,
              batch=19, pf=8.0, pf_lo=1, pf_hi=20, alpha=1.05),
        # 26 one-hot features, skewed queries (workload 2)
        _case("onehot_e64", tables=26, rows_lo=10, rows_hi=4000000, E=64, dtype="f32", max_batch=2048, batch=2048,
              pf=1.0, pf_lo=1, pf_hi=1, alpha=1.05),
        # the same features ranked in bulk with the small row of a compact model
        _case("onehot_bulk_e32", tables=26, rows_lo=10, rows_hi=4000000, E=32, dtype="f32", max_batch=32768,
              batch=32768, pf=1.0, pf_lo=1, pf_hi=1, alpha=1.05),
        # multi-hot features on half-precision tables (workload 3)
        _case("multihot_f16_e128", tables=26, rows_lo=10, rows_hi=4000000, E=128, dtype="f16", max_batch=16384,
              batch=16384, pf=8.0, pf_lo=1, pf_hi=20, alpha=1.0),
        # one table dominates: 50 lookups per query on 10M rows beside 25 one-hot features (workload 4)
        _case("dominant_e64", tables=25, rows_lo=1000, rows_hi=1000000, big_rows=10000000, big_pf=50, big_alpha=1.5,
              E=64, dtype="f32", max_batch=4096, batch=4096, pf=1.0, pf_lo=1, pf_hi=1, alpha=0.0),
        # compact rows, multi-hot, a batch that is no power of two
        _case("multihot_e16", tables=26, rows_lo=10, rows_hi=4000000, E=16, dtype="f32", max_batch=8192, batch=7777,
              pf=8.0, pf_lo=1, pf_hi=20, alpha=1.05),
        # averaged behaviour histories on half-precision rows, some of them empty
        _case("history_mean_f16_e64", tables=40, rows_lo=1000, rows_hi=1000000, E=64, dtype="f16", max_batch=4096,
              batch=4096, pf=4.0, pf_lo=0, pf_hi=10, alpha=1.1, mean=True),
        # weighted multi-hot features
        _case("weighted_e128", tables=32, rows_lo=1000, rows_hi=2000000, E=128, dtype="f32", max_batch=4096,
              batch=3001, pf=20.0, pf_lo=1, pf_hi=100, alpha=1.1, weighted=True),
        # a row width that fills no power of two, long bags without reuse
        _case("long_e96", tables=10, rows_lo=100, rows_hi=3000000, E=96, dtype="f32", max_batch=2048, batch=2048,
              pf=35.0, pf_lo=1, pf_hi=120, alpha=0.0),
        # the widest rows, short averaged bags
        _case("wide_mean_e256", tables=20, rows_lo=1000, rows_hi=1000000, E=256, dtype="f32", max_batch=1000,
              batch=1000, pf=3.0, pf_lo=0, pf_hi=10, alpha=1.05, mean=True),
        # offline scoring, the largest: 100 tables, 131M lookups (workload 5 with its tables cut to the cap)
        _case("bulk_e128", tables=100, rows_lo=1000, rows_hi=2000000, E=128, dtype="f32", max_batch=65536,
              batch=65536, pf=20.0, pf_lo=1, pf_hi=100, alpha=1.1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: every row width, dtype, pooling and option, from one
    query to full batches, of at most a third of the largest listed case's work."""
    dtype = rng.choice(["f32", "f32", "f16"])
    E = rng.choice([16, 24, 32, 48, 64, 96, 100, 128, 200, 256] if dtype == "f32"
                   else [8, 16, 32, 64, 96, 128, 256])
    tables = _log_int(rng, 1, 100)
    rows_lo = _log_int(rng, 10, 2000)
    rows_hi = _log_int(rng, max(rows_lo, 5000), 5000000)
    pf, pf_lo, pf_hi = rng.choice([(1.0, 1, 1), (1.0, 1, 1), (4.0, 0, 10), (8.0, 1, 20), (20.0, 1, 100),
                                   (float(rng.randint(2, 40)), 0, 120)])
    c = _case("", tables=tables, rows_lo=rows_lo, rows_hi=rows_hi, E=E, dtype=dtype,
              pf=pf, pf_lo=pf_lo, pf_hi=pf_hi, alpha=rng.choice([0.0, round(rng.uniform(0.8, 1.5), 2)]),
              mean=rng.random() < 0.3, weighted=rng.random() < 0.25)
    if rng.random() < 0.2:
        c.update(big_rows=_log_int(rng, 1000000, 10000000), big_pf=rng.randint(2, 60),
                 big_alpha=round(rng.uniform(0.8, 1.5), 2))
    per_query = tables * pf + c["big_pf"]
    row_bytes = E * (2 if dtype == "f16" else 4)
    most = min(40e6 / per_query, 22e9 / (per_query * row_bytes), 65536)
    batch = _log_int(rng, 1, max(2, int(most)))
    c["max_batch"] = batch if rng.random() < 0.5 else min(65536, batch + rng.randint(0, batch))
    c["batch"] = batch
    del c["name"]
    return c


def _tables(case):
    """(rows, lookups per bag: mean, least, most, Zipf exponent) of each table."""
    n = case["tables"]
    ratio = case["rows_hi"] / case["rows_lo"]
    rows = [max(1, int(round(case["rows_lo"] * ratio ** (t / (n - 1 if n > 1 else 1))))) for t in range(n)]
    out = [(m, case["pf"], case["pf_lo"], case["pf_hi"], case["alpha"]) for m in rows]
    if case["big_rows"]:
        out.insert(0, (case["big_rows"], float(case["big_pf"]), case["big_pf"], case["big_pf"], case["big_alpha"]))
    row_bytes = case["E"] * (2 if case["dtype"] == "f16" else 4)
    scale = TABLE_BYTES_CAP / max(TABLE_BYTES_CAP, sum(x[0] for x in out) * row_bytes)
    return [(max(1, int(x[0] * scale)),) + x[1:] for x in out]


def _bag_lengths(gen, batch, pf, lo, hi):
    if lo == hi:
        return torch.full((batch,), lo, dtype=torch.int64, device="cuda")
    n = torch.poisson(torch.full((batch,), pf, device="cuda"), generator=gen).to(torch.int64)
    return n.clamp_(lo, hi)


class _Queries:
    """A table's query distribution: bounded Zipf over ranks, a random row for each rank."""

    def __init__(self, gen, rows, alpha):
        self.rows, self.alpha = rows, alpha
        if alpha > 0:
            self.cdf = torch.arange(1, rows + 1, dtype=torch.float64, device="cuda").pow_(-alpha).cumsum_(0)
            self.row_of = torch.randperm(rows, generator=gen, device="cuda")

    def draw(self, gen, n):
        if self.alpha <= 0:
            return torch.randint(0, self.rows, (n,), generator=gen, device="cuda")
        u = torch.rand(n, generator=gen, dtype=torch.float64, device="cuda").mul_(self.cdf[-1])
        return self.row_of[torch.searchsorted(self.cdf, u, right=True).clamp_(max=self.rows - 1)]


def _inputs(case, seed):
    """Tables, indices, offsets and weights of one batch, and the statistics of the queries before it."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dtype = torch.float16 if case["dtype"] == "f16" else torch.float32
    B = case["batch"]
    tables, stats, lengths, indices = [], [], [], []
    for rows, pf, lo, hi, alpha in _tables(case):
        tables.append(torch.empty((rows, case["E"]), dtype=dtype, device="cuda").uniform_(-VALUE, VALUE, generator=gen))
        q = _Queries(gen, rows, alpha)
        past = _bag_lengths(gen, max(1, int(HISTORY_LOOKUPS / pf)), pf, lo, hi)
        ids, counts = torch.unique(q.draw(gen, HISTORY_LOOKUPS), return_counts=True)
        hot = torch.sort(counts, descending=True, stable=True)
        n_hot = min(HOT_LISTED, ids.numel())
        stats.append({"mean_pooling": float(past.double().mean()), "max_pooling": hi,
                      "hot_rows": ids[hot.indices[:n_hot]].cpu().numpy(),
                      "hot_freq": hot.values[:n_hot].double().cpu().numpy() / HISTORY_LOOKUPS,
                      "unique_frac": ids.numel() / HISTORY_LOOKUPS})
        n = _bag_lengths(gen, B, pf, lo, hi)
        lengths.append(n)
        indices.append(q.draw(gen, int(n.sum())))
    offsets = torch.zeros(len(tables) * B + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cat(lengths).cumsum(0)
    indices = torch.cat(indices)
    weights = torch.rand(indices.numel(), generator=gen, device="cuda").add_(0.5) if case["weighted"] else None
    return tables, stats, indices, offsets, weights


def prepare(case, seed):
    tables, stats, indices, offsets, weights = _inputs(case, seed)
    plan = embx.Plan([w.shape[0] for w in tables], case["E"], case["dtype"], stats, case["max_batch"],
                     pooling="mean" if case["mean"] else "sum").bind(tables)
    out = torch.empty((case["batch"], len(tables), case["E"]), dtype=torch.float32, device="cuda")
    return plan, indices, offsets, case["batch"], out, weights


def run(state):
    plan, indices, offsets, batch, out, weights = state
    return plan.lookup(indices, offsets, batch, out, weights=weights)


def _distinct(rows, n, alpha):
    """Expected distinct rows among n lookups of a table (ranks taken in geometric bins)."""
    if alpha <= 0:
        return rows * -math.expm1(-n / rows)
    edge = np.unique(np.round(np.geomspace(1, rows + 1, 2000)).astype(np.int64))
    width = np.diff(edge)
    rank = np.sqrt(edge[:-1].astype(np.float64) * np.maximum(edge[1:] - 1, 1))
    p = rank ** -alpha
    p /= (p * width).sum()
    return float((width * -np.expm1(-n * p)).sum())


def work(case):
    """Each distinct row, index, weight and offset read once, each pooled output written once;
    an addition per looked-up element (a multiplication more with weights)."""
    E, B = case["E"], case["batch"]
    row_bytes = E * (2 if case["dtype"] == "f16" else 4)
    tables = _tables(case)
    lookups = rows = 0.0
    for m, pf, lo, hi, alpha in tables:
        lookups += B * pf
        rows += _distinct(m, B * pf, alpha)
    total = rows * row_bytes + lookups * (12 if case["weighted"] else 8) + (len(tables) * B + 1) * 8 \
        + len(tables) * B * E * 4
    return {"bytes": total, "flops": lookups * E * (2 if case["weighted"] else 1)}


def tolerance(case):
    # fp32 sums of up to 120 terms (measured against ``exact``: 0 to 8.4e-8)
    return {"rel": 4e-7, "max": 4e-6}


def exact(case, seed):
    tables, _, indices, offsets, weights = _inputs(case, seed)
    B = case["batch"]
    out = torch.empty((B, len(tables), case["E"]), dtype=torch.float64, device="cuda")
    ends = offsets[::B].tolist()   # where each table's lookups start
    for t, w in enumerate(tables):
        rows, local = torch.unique(indices[ends[t]:ends[t + 1]], return_inverse=True)
        if rows.numel() == 0:
            out[:, t] = 0.0
            continue
        vals = w[rows].double()
        psw = weights[ends[t]:ends[t + 1]].double() if weights is not None else None
        bags = F.embedding_bag(local, vals, offsets[t * B:(t + 1) * B] - ends[t], mode="sum", per_sample_weights=psw)
        if case["mean"]:
            n = (offsets[t * B + 1:(t + 1) * B + 1] - offsets[t * B:(t + 1) * B]).clamp(min=1)
            bags = bags / n.double()[:, None]
        out[:, t] = bags
    return out
