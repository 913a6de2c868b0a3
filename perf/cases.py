"""The measured workloads of the table-batched embedding step, through the public entry points.

A case names the tables, the batch, the element types and the calls of one pass:

  op       forward | backward | step (forward + backward) | seq (non-pooled lookup + its backward) | sync (replica mean)
  tables   groups "COUNTxROWSxWIDTHS", joined by "+"; ROWS is a number or "lo-hi" (spread evenly over the logarithm),
           WIDTHS one or more columns counts taken in turn, "128/256/256"
  weights  f32 | f16            ids  i64 | i32 (ids and offsets)          io  f32 | f16 | bf16 (pooled output and gradient)
  B        samples per batch; every table has one bag per sample
  lengths  "fixed L" | "poisson L" (bags may be empty) | "poisson1 L" (one more than Poisson) | "lognormal mu sigma cap"
  zipf     exponent of the ids' popularity, 0: uniform
  update   adagrad | static (the library's own scratch) | split (prepare, then apply) | sgd
"""
import math

import numpy as np
import torch

from paper_2508_03854_amd import TBE

LR, SGD_LR, EPS = 0.01, 1e-4, 1e-8
_IDX = {"i64": torch.int64, "i32": torch.int32}
_IO = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_BYTES = {"i64": 8, "i32": 4, "f32": 4, "f16": 2, "bf16": 2}


def _pooled(name, op, tables, B, lengths, zipf, weights="f32", ids="i64", io="f32", pooling="sum", update="adagrad", c=1.0):
    return {"name": name, "op": op, "tables": tables, "B": B, "lengths": lengths, "zipf": zipf, "weights": weights,
            "ids": ids, "io": io, "pooling": pooling, "update": update, "c": c}


def listed():
    return [
        # a single request in a serving loop: a handful of features, a few samples, latency only
        _pooled("serve_request", "forward", "8x100000x64", 32, "poisson1 10", 1.05),
        # candidates of a ranking service over half-precision tables: no backward, so nothing is known of the hot rows
        _pooled("serve_ranking", "forward", "64x10000-1000000x128/256/256/256", 3001, "poisson1 30", 1.1, weights="f16",
                ids="i32", io="f16"),
        # the smallest training step: one table, uniform ids, a chain of small launches
        _pooled("step_one_table", "step", "1x100000x64", 512, "fixed 20", 0.0),
        # odd widths on both sides of every width class, ragged batch, empty bags, the backward that allocates nothing
        _pooled("step_odd_widths", "step", "10x700-90000x20/36/100/12/260/64/516/132/8/1024", 777, "poisson 6", 1.2,
                ids="i32", io="f16", pooling="mean", update="static", c=2.0),
        # a public click-log model's tables: 26 features of one width
        _pooled("step_26_tables", "step", "26x1000-1000000x64", 4096, "poisson1 10", 1.05),
        # several widths and very different table sizes, strong skew: many duplicates on few rows
        _pooled("step_mixed_widths", "step", "16x10000-10000000x64/128/256", 16384, "poisson1 20", 1.2, c=4.0),
        # a quarter of a production shard at its full batch: half-precision rows, fp32 moments
        _pooled("step_production", "step", "64x25000-2500000x128/256/256/256", 32768, "poisson1 30", 1.1, weights="f16"),
        # the same kind of shard at the batch per GPU of a large job, narrow streams, sort split off the critical path
        _pooled("step_narrow_streams", "step", "64x25000-2500000x128/256/256/256", 4096, "poisson1 30", 1.1, weights="f16",
                ids="i32", io="bf16", update="split"),
        # the straggler: two large tables among small narrow ones, long-tailed bags, mean pooling, very hot rows
        _pooled("step_straggler", "step", "2x5000000x128+30x100000x32", 65536, "lognormal 2 1 500", 1.3, pooling="mean"),
        # cold ids: nearly every lookup its own row, so the row update itself is what counts
        _pooled("backward_cold_ids", "backward", "12x1000000x128", 8192, "fixed 20", 0.0),
        # sequence features: one row per event, its gradient per event
        _pooled("sequence_events", "seq", "2x2000000x128+14x100000x32", 16000, "lognormal 2 1 500", 1.3, io="bf16"),
        # the weight sync of four replicas held on one device
        {"name": "replica_sync", "op": "sync", "replicas": 4, "count": 60_000_012, "weights": "f32"},
    ]


def draw(rng):
    def spread(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    op = rng.choice(("forward", "forward", "step", "step", "step", "step", "backward", "seq", "sync"))
    if op == "sync":
        weights = rng.choice(("f32", "f16"))
        m = rng.choice((2, 3, 4, 8))
        return {"op": op, "replicas": m, "count": 4 * int(spread(5_000, 80_000_000 // m)) + rng.randrange(4), "weights": weights}
    weights = rng.choice(("f32", "f32", "f16"))
    ids = rng.choice(("i64", "i64", "i32"))
    io = rng.choice(("f32", "f32", "f16", "bf16"))
    widths = rng.choice(("32", "64", "64", "128", "64/128/256", "128/256/256/256", "256", "24/40/104/8/264/136/520"))
    mean_width = sum(map(int, widths.split("/"))) / len(widths.split("/"))
    T = max(1, min(64, round(spread(1, 70))))
    B = max(1, min(65536, round(spread(24, 80_000))))
    length = spread(3, 35)
    zipf = rng.choice((0.0, 1.05, 1.1, 1.2, 1.3))
    most = 6.0e9 if op in ("forward", "backward") else 4.0e9      # gathered elements of one pass
    while T * B * length * mean_width > most or B * T * mean_width > 4.0e8:
        T, B = (max(1, T * 2 // 3), B) if rng.random() < 0.5 else (T, B * 2 // 3)
    hi = spread(20_000, max(40_000, min(5_000_000, 3.0e9 / (T * mean_width))))
    lo = max(500, hi / spread(1, 300))
    rows = "%d-%d" % (lo, hi) if rng.random() < 0.8 else "%d" % hi
    lengths = rng.choice(("fixed %d" % round(length), "poisson %.1f" % length, "poisson1 %.1f" % length, "poisson1 %.1f" % length,
                          "lognormal %.2f 1 500" % (math.log(length) - 0.5)))
    if op == "seq":
        pooling, update = "sum", "adagrad"
    else:
        pooling = rng.choice(("sum", "sum", "mean"))
        small = T * B * length < 250_000 and T * 1024 * mean_width < 6_000_000
        update = rng.choice(("adagrad", "adagrad", "split", "sgd", "static" if small else "adagrad"))
    c = rng.choice((1.0, 2.0, 4.0))
    case = _pooled("", op, "%dx%sx%s" % (T, rows, widths), B, lengths, zipf, weights, ids, io, pooling, update, c)
    del case["name"]
    return case


def _tables(case):
    """(rows, widths) of every table."""
    rows, widths = [], []
    for group in case["tables"].split("+"):
        count, r, w = group.split("x")
        w = [int(x) for x in w.split("/")]
        lo, hi = (float(x) for x in (r.split("-") if "-" in r else (r, r)))
        for t in range(int(count)):
            at = (0.5 + t * 0.6180339887498949) % 1.0
            rows.append(max(4, round(lo * (hi / lo) ** at)))
            widths.append(w[t % len(w)])
    return rows, widths


def _mean_length(case):
    kind, *p = case["lengths"].split()
    p = [float(x) for x in p]
    return p[0] if kind in ("fixed", "poisson") else p[0] + 1.0 if kind == "poisson1" else math.exp(p[0] + 0.5 * p[1] * p[1])


def _lookups(case, T):
    """Lookups per table: what the bags hold on average, or for sequences the very number of events."""
    n = case["B"] * _mean_length(case)
    return [int(n * (0.75 + 0.5 * ((0.25 + t * 0.6180339887498949) % 1.0))) for t in range(T)] if case["op"] == "seq" else [n] * T


def _distinct(n, R, s):
    """Expected number of distinct rows among n lookups of a table of R rows."""
    if s == 0.0:
        return -R * math.expm1(-n / R)
    edge = np.arange(0, R + 1, dtype=np.float64) + 0.5
    f = edge ** (1.0 - s)
    p = (f[:-1] - f[1:]) / (f[0] - f[-1])
    return float(-np.expm1(-n * p).sum())


def work(case):
    w = _BYTES[case["weights"]]
    if case["op"] == "sync":
        return {"bytes": 2 * case["replicas"] * case["count"] * w, "flops": case["replicas"] * case["count"]}
    rows, D = _tables(case)
    ib, eb = _BYTES[case["ids"]], _BYTES[case["io"]]
    n = _lookups(case, len(D))
    U = [_distinct(m, r, case["zipf"]) for m, r in zip(n, rows)]
    row_bytes = sum(u * d * w for u, d in zip(U, D))
    ids = (sum(n) + len(D) * (1 if case["op"] == "seq" else case["B"])) * ib
    adds = sum(m * d for m, d in zip(n, D))
    dense = (adds if case["op"] == "seq" else case["B"] * sum(D)) * eb
    moments = 0 if case["update"] == "sgd" else 8 * sum(U)
    if case["op"] == "forward":
        return {"bytes": ids + row_bytes + dense, "flops": adds}
    # the distinct rows are read and written once, their moments too; ids, offsets, output and gradient pass once
    backward = ids + dense + 2 * row_bytes + moments
    return {"bytes": backward if case["op"] == "backward" else backward + dense, "flops": adds * (1 if case["op"] == "backward" else 2)}


def tolerance(case):
    if case["op"] == "sync":
        return {"rel": 1e-6 if case["weights"] == "f32" else 1e-3}
    # 16-bit values: two correct sums may round to neighbours
    return {"rel": 1e-2 if case["io"] == "bf16" else 2e-3 if "f16" in (case["io"], case["weights"]) else 1e-5}


def _lengths(case, n, g):
    kind, *p = case["lengths"].split()
    p = [float(x) for x in p]
    if kind == "fixed":
        return torch.full((n,), int(p[0]), dtype=torch.int64, device="cuda")
    if kind == "lognormal":
        z = torch.randn(n, generator=g, device="cuda")
        return torch.round(torch.exp(p[0] + p[1] * z)).to(torch.int64).clamp_(1, int(p[2]))
    lam = torch.full((n,), p[0], device="cuda")
    return torch.poisson(lam, generator=g).to(torch.int64) + (1 if kind == "poisson1" else 0)


def _ids(rows, per_table, s, g):
    """Table-local ids in table order: bounded Zipf(s) by inverse distribution function, the popular rows scattered over
    the table by a multiplication modulo its size."""
    dev = "cuda"
    step = []
    for r in rows:
        a = int(r * 0.6180339887498949) | 1
        while math.gcd(a, r) != 1:
            a += 1
        step.append(a % r if r > 1 else 0)
    t = torch.repeat_interleave(torch.arange(len(rows), device=dev), per_table)
    R = torch.tensor(rows, dtype=torch.int64, device=dev)[t]
    u = torch.rand(t.numel(), generator=g, dtype=torch.float64, device=dev)
    if s == 0.0:
        return torch.minimum((u * R).to(torch.int64), R - 1)
    lo = 0.5 ** (1.0 - s)
    hi = (R.to(torch.float64) + 0.5).pow_(1.0 - s)
    rank = torch.round((lo - u * (lo - hi)).pow_(1.0 / (1.0 - s))).to(torch.int64)
    rank = torch.minimum(rank.clamp_(min=1), R) - 1
    return (rank * torch.tensor(step, dtype=torch.int64, device=dev)[t]) % R


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["op"] == "sync":
        dt = _IO[case["weights"]]
        reps = [torch.empty(case["count"], dtype=dt, device="cuda").uniform_(-0.01, 0.01, generator=g)
                for _ in range(case["replicas"])]
        return {"case": case, "tbe": TBE([16], [8], case["weights"]), "replicas": reps}
    rows, D = _tables(case)
    T, B, seq = len(rows), case["B"], case["op"] == "seq"
    if seq:
        L = per_table = torch.tensor(_lookups(case, T), dtype=torch.int64, device="cuda")
    else:
        L = _lengths(case, T * B, g)
        per_table = L.view(T, B).sum(1)
    idx = _ids(rows, per_table, case["zipf"], g)
    off = torch.zeros(L.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(L, 0, out=off[1:])
    it, io = _IDX[case["ids"]], _IO[case["io"]]
    tbe = TBE(rows, D, case["weights"])
    dense = (int(sum(n * d for n, d in zip(per_table.tolist(), D))),) if seq else (B, tbe.sum_D)
    s = {"case": case, "tbe": tbe, "B": B, "idx": idx.to(it), "off": off.to(it), "nnz": idx.numel(),
         "tables": torch.empty(tbe.total_elems, dtype=tbe.torch_dtype, device="cuda").uniform_(-0.01, 0.01, generator=g)}
    if case["op"] != "backward":
        s["out"] = torch.empty(dense, dtype=io, device="cuda")
    if case["op"] != "forward":
        s["grad"] = torch.randn(dense, generator=g, device="cuda").to(io)
        if case["update"] != "sgd":
            s["state"] = torch.rand(tbe.total_rows, generator=g, device="cuda").mul_(4.0).add_(1e-3)
        if case["update"] != "static":
            s["workspace"] = tbe.alloc_workspace(1 if seq else B, s["nnz"])
    return s


def _backward(s):
    case, tbe, B = s["case"], s["tbe"], s["B"]
    step = {"pooling": case["pooling"], "lr": SGD_LR if case["update"] == "sgd" else LR}
    adagrad = dict(step, eps=EPS, momentum_scale=case["c"])
    if case["update"] == "sgd":
        tbe.backward_sgd(s["grad"], s["idx"], s["off"], B, s["tables"], s["workspace"], **step)
    elif case["update"] == "static":
        tbe.backward_rowwise_adagrad_static(s["grad"], s["idx"], s["off"], B, s["tables"], s["state"], **adagrad)
    elif case["update"] == "split":
        tbe.backward_prepare(s["idx"], s["off"], B, s["workspace"])
        tbe.backward_apply_rowwise_adagrad(s["grad"], s["off"], B, s["nnz"], s["tables"], s["state"], s["workspace"], **adagrad)
    elif case["ids"] == "i64" and case["io"] == "f32":
        tbe.backward_rowwise_adagrad(s["grad"], s["idx"], s["off"], B, s["tables"], s["state"], s["workspace"], **adagrad)
    else:
        tbe.backward_rowwise_adagrad_ex(s["grad"], s["idx"], s["off"], B, s["tables"], s["state"], s["workspace"], **adagrad)


def run(s):
    case, tbe = s["case"], s["tbe"]
    if case["op"] == "sync":
        tbe.replica_mean(s["replicas"])
        return s["replicas"]
    if case["op"] == "seq":
        tbe.lookup_seq(s["tables"], s["idx"], s["off"], s["out"])
        tbe.backward_seq_rowwise_adagrad(s["grad"], s["idx"], s["off"], s["tables"], s["state"], s["workspace"], lr=LR, eps=EPS,
                                         momentum_scale=case["c"])
    else:
        if case["op"] != "backward":
            if case["ids"] == "i64" and case["io"] == "f32":
                tbe.forward(s["tables"], s["idx"], s["off"], s["B"], case["pooling"], out=s["out"])
            else:
                tbe.forward_ex(s["tables"], s["idx"], s["off"], s["B"], case["pooling"], out=s["out"])
        if case["op"] != "forward":
            _backward(s)
    if case["op"] == "forward":
        return s["out"]
    return {k: s[k] for k in ("out", "tables", "state") if k in s}
