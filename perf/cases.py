"""Performance cases of the library: what a recommender or a tensor-parallel
layer calls, over the sizes, types and options it is called with.

A case is one call sequence of the public Python binding
(``paper_2305_06942_amd``) on device buffers the caller already holds:

* ``forward``: fused embedding-bag pooling into the All-to-All send layout;
* ``forward_consume``: the same with the consumer draining finished slices on
  a second hardware queue (the whole operator as a training step runs it);
* ``unfused``, ``noalloc``: the bulk-synchronous and the plan-free forward;
* ``backward``: one gradient row per lookup from the pooled gradient;
* ``deliver_backward``: the gradient's arrival on one queue, the backward
  expanding each slice as its flag lands on another;
* ``gemv``: the fused GEMV + AllReduce of a tensor-parallel layer.

Table values are U(-0.05, 0.05) as embedding tables are initialised, indices
uniform or Zipf-distributed over scattered rows, bag lengths fixed, uniform or
clipped Poisson, weights U[0, 1), gradients and activations normal.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2305_06942_amd as ebag

DEV = "cuda"
TORCH_TYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
ABI_TYPE = {"f32": 0, "f16": 1, "bf16": 2}
ELT = {"f32": 4, "f16": 2, "bf16": 2}


def _bags(name, kind, T, rows, dims, dtype, B, R, C, lengths, indices="uniform", pooling="sum", opts=""):
    """dims: comma list, cycled over the T tables; opts: 'name=value,...' of the plan."""
    return {"name": name, "kind": kind, "T": T, "rows": rows, "dims": dims, "dtype": dtype, "B": B, "R": R, "C": C,
            "lengths": lengths, "indices": indices, "pooling": pooling, "opts": opts}


def _gemv(name, R, M, K, dtype):
    """K: comma list of the ranks' columns (one value: every rank)."""
    return {"name": name, "kind": "gemv", "R": R, "M": M, "K": K, "dtype": dtype}


def listed():
    return [
        # A small serving call (the "tiny" workload): launch latency and host work decide.
        _bags("fwd_tiny", "forward", 4, 10_000, "64", "f32", 256, 2, 32, "fixed:8"),
        # One-hot and few-hot categorical features, some absent: 26 tables, 0 to 3 lookups a bag.
        _bags("fwd_short_bags", "forward", 26, 1_000_000, "128", "f32", 16384, 8, 64, "uniform:0:3"),
        # The whole operator on the "dlrm" workload: pooling with the consumer draining slices behind it.
        _bags("fwd_consume_dlrm", "forward_consume", 32, 1_000_000, "128", "f32", 4096, 8, 64, "fixed:32"),
        # The "skewed" workload: fp16 tables, Zipf(1.05) indices, in its own launch options.
        _bags("fwd_skewed_f16", "forward", 64, 500_000, "256", "f16", 8192, 8, 64, "uniform:1:64", "zipf:1.05", "sum",
              "stream_rows=0,table_major=1,slice_granule=1,waves_per_wg=2,bags_per_run=8"),
        # The headline "large" workload at a quarter of its tables, so that three states fit the card.
        _bags("fwd_large_f32", "forward", 32, 2_000_000, "128", "f32", 16384, 64, 32, "poisson:40:1:128", "zipf:0.9",
              "sum", "stream_rows=0,table_major=2,slice_granule=1,bags_per_run=8"),
        # The "mixed" workload: bf16 tables of four widths, long ragged bags, per-lookup weights.
        _bags("fwd_mixed_bf16", "forward", 48, 1_000_000, "32,64,128,256", "bf16", 8192, 16, 128, "uniform:1:100",
              "uniform", "weighted", "stream_rows=0,table_major=2,slice_granule=1"),
        # Widths that are no power of two (rows of 6, 12, 20 and 40 sixteen-byte vectors), a batch split in three,
        # slices of 50 samples: default options.
        _bags("fwd_odd_widths", "forward", 24, 500_000, "48,96,160,320", "f16", 6150, 3, 50, "uniform:1:40"),
        # Tables above 4 GiB (10 M rows of 512 bytes), mean pooling: default options.
        _bags("fwd_big_tables_mean", "forward", 4, 10_000_000, "128", "f32", 16384, 8, 64, "uniform:1:40", "uniform",
              "mean"),
        # Embedding backward of the "mixed" workload, gradient complete: weighted, ragged.
        _bags("bwd_mixed_weighted", "backward", 48, 1_000_000, "32,64,128,256", "bf16", 8192, 16, 128,
              "uniform:1:100", "uniform", "weighted", "table_major=2,slice_granule=1,backward_bags_per_run=8"),
        # Embedding backward overlapped with the gradient's arrival, on the "dlrm" workload.
        _bags("bwd_deliver_dlrm", "deliver_backward", 32, 1_000_000, "128", "f32", 4096, 8, 64, "fixed:32"),
        # A 4096 x 4096 projection split over eight ranks, one token: the smallest layer call.
        _gemv("gemv_4096_bf16", 8, 4096, "512", "bf16"),
        # The benchmark's largest GEMV + AllReduce.
        _gemv("gemv_65536_f16", 4, 65536, "2048", "f16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Most bytes of lookups, outputs or tables that a drawn case may ask for.
_MOST_BYTES = 5e9
_MOST_TABLE_BYTES = 12e9


def draw(rng):
    """One more case over the same ranges: every call, storage type, pooling
    mode and option, widths of one to 64 sixteen-byte vectors, odd batches."""
    dtype = rng.choice(("f32", "f16", "bf16"))
    elt = ELT[dtype]
    kind = rng.choice(("forward", "forward", "forward", "forward", "forward_consume", "unfused", "noalloc", "backward",
                       "backward", "deliver_backward", "gemv", "gemv"))
    if kind == "gemv":
        R = rng.choice((1, 2, 4, 8, 16))
        M = _log_int(rng, 256, 65536)
        K = [min(65536 // elt, _log_int(rng, 64, 8192)) // 8 * 8 for _ in range(R if rng.random() < 0.3 else 1)]
        while M * sum(K) * (R // len(K)) * elt > 1.2e9:
            M = M // 2 + 1
        return {"kind": kind, "R": R, "M": M, "K": ",".join(map(str, K)), "dtype": dtype}
    vecs = [rng.choice((1, 2, 3, 4, 5, 6, 8, 8, 12, 16, 16, 20, 24, 32, 32, 40, 48, 64))
            for _ in range(rng.choice((1, 1, 1, 2, 3, 4)))]
    dims = [v * 16 // elt for v in vecs]
    T = _log_int(rng, 1, 64)
    row_bytes = sum(dims[t % len(dims)] for t in range(T)) * elt
    rows = _log_int(rng, 1000, max(1000, min(4_000_000, int(_MOST_TABLE_BYTES / row_bytes))))
    lengths = rng.choice(("fixed:1", "uniform:0:3", "uniform:1:40", "uniform:1:100", "fixed:32", "poisson:40:1:128",
                          "uniform:1:64"))
    R = rng.choice((1, 2, 3, 4, 8, 16))
    C = rng.choice((16, 25, 32, 50, 64, 128))
    B = R * C * max(1, _log_int(rng, 64, 16384) // (R * C))
    widest = 4 if "backward" in kind else elt  # the backward writes fp32 rows
    while B > R * C and B * row_bytes // elt * (widest * _mean_length(lengths) + 8) > _MOST_BYTES:
        B = R * C * max(1, B // (2 * R * C))
    pooling = rng.choice(("sum", "sum", "weighted", "mean"))
    opts = rng.choice(("", "", "", "stream_rows=0,table_major=1,slice_granule=1", "stream_rows=0,table_major=2,slice_granule=1",
                       "persistent_wgs_per_cu=-1", "chunk_order=1", "check_indices=1"))
    if kind == "noalloc" and opts == "check_indices=1":
        opts = ""
    case = _bags("", kind, T, rows, ",".join(map(str, dims)), dtype, B, R, C, lengths,
                 rng.choice(("uniform", "uniform", "zipf:0.9", "zipf:1.05")), pooling, opts)
    del case["name"]
    return case


# ------------------------------------------------------------------ inputs

def _dims(case):
    d = [int(x) for x in case["dims"].split(",")]
    return [d[t % len(d)] for t in range(case["T"])]


def _opts(case):
    o = {k: int(v) for k, v in (kv.split("=") for kv in case["opts"].split(",") if kv)}
    if case["pooling"] == "mean":
        o["pooling_mode"] = 1
    return o


def _gemv_k(case):
    K = [int(x) for x in case["K"].split(",")]
    return K * case["R"] if len(K) == 1 else K


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _mean_length(law):
    kind, *p = law.split(":")
    p = [float(x) for x in p]
    return (p[0] + p[1]) / 2 if kind == "uniform" else p[0]


def _draw_lengths(law, T, B, g):
    """Bag lengths [T, B]: each table's are one sample of the law, put in an
    order of the seed's own, so that every seed has as many lookups and the
    outputs the same sizes."""
    kind, *p = law.split(":")
    p = [int(x) for x in p]
    if kind == "fixed":
        return torch.full((T, B), p[0], dtype=torch.int64, device=DEV)
    same = _generator(1)
    if kind == "uniform":
        lengths = torch.randint(p[0], p[1] + 1, (T, B), generator=same, device=DEV)
    else:
        lengths = torch.poisson(torch.full((T, B), float(p[0]), device=DEV), generator=same).long().clamp_(p[1], p[2])
    return lengths.gather(1, torch.rand((T, B), generator=g, device=DEV).argsort(1))


@functools.lru_cache(maxsize=4)
def _zipf_p(n, alpha):
    w = np.arange(1, n + 1, dtype=np.float64) ** (-alpha)
    return w / w.sum()


def _draw_indices(law, bounds, rows, g, seed):
    """int32 indices of every table; bounds: first lookup of each table and
    the end.  Zipf ranks are scattered over the table by r -> (a r + b) mod
    rows, a bijection of the rows."""
    n = bounds[-1]
    if law == "uniform":
        return torch.randint(0, rows, (n,), generator=g, device=DEV, dtype=torch.int32)
    cdf = torch.from_numpy(np.cumsum(_zipf_p(rows, float(law.split(":")[1])))).to(DEV)
    idx = torch.empty(n, dtype=torch.int32, device=DEV)
    r = np.random.default_rng([seed, 7])
    for lo, hi in zip(bounds[:-1], bounds[1:]):
        rank = torch.searchsorted(cdf, torch.rand(hi - lo, generator=g, device=DEV, dtype=torch.float64), right=True)
        a = int(r.integers(1, rows + 1))
        while math.gcd(a, rows) != 1:
            a += 1
        idx[lo:hi] = ((rank.clamp_(max=rows - 1) * a + int(r.integers(0, rows))) % rows).int()
    return idx


def _bag_inputs(case, seed, tables):
    """Bags (and, for a forward, tables; for a backward, the gradient)."""
    g = _generator(seed)
    T, B, dims = case["T"], case["B"], _dims(case)
    lengths = _draw_lengths(case["lengths"], T, B, g)
    offsets = torch.zeros(T * B + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lengths.view(-1), 0, out=offsets[1:])
    bounds = offsets[::B].tolist()
    s = {"offsets": offsets, "bounds": bounds, "weights": None}
    if case["pooling"] == "weighted":
        s["weights"] = torch.rand(bounds[-1], generator=g, device=DEV)
    if tables:
        s["indices"] = _draw_indices(case["indices"], bounds, case["rows"], g, seed)
        s["tables"] = [torch.empty((case["rows"], d), device=DEV).uniform_(-0.05, 0.05, generator=g)
                       .to(TORCH_TYPE[case["dtype"]]) for d in dims]
    else:
        s["grad"] = torch.randn((B, sum(dims)), generator=g, device=DEV)
    return s


def _gemv_inputs(case, seed):
    g = _generator(seed)
    dt = TORCH_TYPE[case["dtype"]]
    K = _gemv_k(case)
    scale = sum(K) ** -0.5
    A = [torch.randn((case["M"], k), generator=g, device=DEV).mul_(scale).to(dt) for k in K]
    x = [torch.randn((k,), generator=g, device=DEV).to(dt) for k in K]
    return A, x


_QUEUES = []


def _queues():
    """The two hardware queues a program overlaps producer and consumer on."""
    if not _QUEUES:
        _QUEUES.extend((ebag.queue_stream(), ebag.queue_stream()))
    return _QUEUES


def prepare(case, seed):
    if case["kind"] == "gemv":
        A, x = _gemv_inputs(case, seed)
        plan = ebag.GemvAR(case["R"], case["M"], _gemv_k(case), ABI_TYPE[case["dtype"]])
        return {"case": case, "plan": plan, "A": A, "x": x,
                "y": [torch.empty(case["M"], device=DEV) for _ in A],
                "flags": torch.zeros(case["R"] * plan.launch_info()[0], dtype=torch.int32, device=DEV)}
    kind, B, R, C, dims = case["kind"], case["B"], case["R"], case["C"], _dims(case)
    backward = "backward" in kind
    s = _bag_inputs(case, seed, not backward)
    s.update(case=case, epoch=0, opts=_opts(case), rows=[case["rows"]] * case["T"], dims=dims)
    per_table = case["T"] if s["opts"].get("slice_granule") == 1 else 1
    if kind != "noalloc":
        s["plan"] = ebag.Plan(s["rows"], dims, ABI_TYPE[case["dtype"]], C, B, R, **s["opts"])
    s["flags"] = torch.zeros(B // C * per_table, dtype=torch.int32, device=DEV)
    if kind in ("forward_consume", "deliver_backward"):
        _queues()
        s["recv"] = torch.empty((B, sum(dims)), device=DEV)
    if backward:
        bounds = s["bounds"]
        s["values"] = torch.empty(sum((bounds[t + 1] - bounds[t]) * d for t, d in enumerate(dims)), device=DEV)
    else:
        s["send"] = torch.empty((B, sum(dims)), device=DEV)
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "gemv":
        s["plan"].forward(s["A"], s["x"], s["y"], s["flags"])
        return {"y": s["y"], "flags": s["flags"]}
    B, R = case["B"], case["R"]
    s["epoch"] += 1
    if kind == "forward":
        s["plan"].forward(s["tables"], s["indices"], s["offsets"], s["weights"], B, R, s["send"], s["flags"])
        return {"send": s["send"], "flags": s["flags"]}
    if kind == "unfused":
        s["plan"].unfused_forward(s["tables"], s["indices"], s["offsets"], s["weights"], B, R, s["send"], s["flags"])
        return {"send": s["send"], "flags": s["flags"]}
    if kind == "noalloc":
        ebag.forward_noalloc(s["rows"], s["dims"], ABI_TYPE[case["dtype"]], case["C"], s["tables"], s["indices"],
                             s["offsets"], s["weights"], B, R, s["send"], s["flags"], **s["opts"])
        return {"send": s["send"], "flags": s["flags"]}
    if kind == "backward":
        s["plan"].backward(s["grad"], s["offsets"], s["weights"], B, R, s["values"])
        return {"values": s["values"]}
    prod, cons = _queues()
    main = torch.cuda.current_stream()
    prod.wait_stream(main)
    cons.wait_stream(main)
    if kind == "forward_consume":  # producer first: the consumer can never be queued ahead of it
        s["plan"].forward(s["tables"], s["indices"], s["offsets"], s["weights"], B, R, s["send"], s["flags"],
                          stream=prod)
        s["plan"].consume(s["send"], s["flags"], s["recv"], B, R, s["epoch"], stream=cons)
        out = {"send": s["send"], "recv": s["recv"], "flags": s["flags"]}
    else:
        s["plan"].deliver(s["grad"], s["recv"], s["flags"], B, R, stream=prod)
        s["plan"].backward(s["recv"], s["offsets"], s["weights"], B, R, s["values"], grad_flags=s["flags"],
                           expected_epoch=s["epoch"], stream=cons)
        out = {"values": s["values"], "recv": s["recv"], "flags": s["flags"]}
    main.wait_stream(prod)
    main.wait_stream(cons)
    return out


# ------------------------------------------------------------------ what a pass cannot do without

def _distinct_rows(law, n, rows):
    """Expected distinct rows of n lookups into a table of `rows` rows."""
    if law == "uniform":
        return -rows * math.expm1(n * math.log1p(-1.0 / rows)) if rows > 1 else min(n, 1)
    p = np.minimum(_zipf_p(rows, float(law.split(":")[1])), 1 - 1e-12)
    return float(-np.expm1(n * np.log1p(-p)).sum())


def work(case):
    elt = ELT[case["dtype"]]
    if case["kind"] == "gemv":
        K, M = sum(_gemv_k(case)), case["M"]
        return {"bytes": M * K * elt + K * elt + 4 * case["R"] * M, "flops": 2 * M * K}
    T, B, dims = case["T"], case["B"], _dims(case)
    n = B * _mean_length(case["lengths"])  # lookups of one table
    pooled = 4 * B * sum(dims)
    csr = 8 * (T * B + 1) + (4 * T * n if case["pooling"] == "weighted" else 0)
    weighted = 2 if case["pooling"] == "weighted" else 1
    if "backward" in case["kind"]:
        moved = 3 * pooled if case["kind"] == "deliver_backward" else pooled  # arrival: read and written once more
        return {"bytes": moved + csr + 4 * n * sum(dims), "flops": (weighted - 1) * n * sum(dims)}
    rows = _distinct_rows(case["indices"], n, case["rows"]) * sum(dims) * elt
    moved = 2 * pooled if case["kind"] == "forward_consume" else pooled
    return {"bytes": rows + 4 * T * n + csr + moved, "flops": weighted * n * sum(dims)}


def tolerance(case):
    if "backward" in case["kind"]:
        return "exact"  # one multiply or divide per value, rounded once
    # fp32 sums of up to 128 rows, or over a rank's columns and the ranks: 0.3e-7 to 1.3e-7 off exact() as measured
    return {"rel": 5e-7}


# ------------------------------------------------------------------ the same in 64 bits

def exact(case, seed):
    if case["kind"] == "gemv":
        A, x = _gemv_inputs(case, seed)
        y = torch.zeros(case["M"], dtype=torch.float64, device=DEV)
        for a, v in zip(A, x):
            for r in range(0, case["M"], 8192):
                y[r:r + 8192] += (a[r:r + 8192].double() * v.double()).sum(1)
        return {"y": [y] * case["R"], "flags": None}
    backward = "backward" in case["kind"]
    s = _bag_inputs(case, seed, not backward)
    T, B, dims, bounds = case["T"], case["B"], _dims(case), s["bounds"]
    lengths = s["offsets"].diff().view(T, B)
    out, col = [], 0
    for t, d in enumerate(dims):
        bag = torch.repeat_interleave(torch.arange(B, device=DEV), lengths[t])
        lo, hi = bounds[t], bounds[t + 1]
        count = lengths[t].clamp(min=1).double()
        if backward:
            v = s["grad"][:, col:col + d].double()[bag]
            if s["weights"] is not None:
                v *= s["weights"][lo:hi].double()[:, None]
            if case["pooling"] == "mean":
                v /= count[bag][:, None]
            out.append(v.reshape(-1))
        else:
            v = s["tables"][t][s["indices"][lo:hi].long()].double()
            if s["weights"] is not None:
                v *= s["weights"][lo:hi].double()[:, None]
            p = torch.zeros((B, d), dtype=torch.float64, device=DEV).index_add_(0, bag, v)
            out.append(p / count[:, None] if case["pooling"] == "mean" else p)
        col += d
        del v
    if backward:
        res = {"values": torch.cat(out)}
        if case["kind"] == "deliver_backward":
            res.update(recv=s["grad"].double(), flags=None)
        return res
    pooled = torch.cat(out, 1)
    if case["kind"] == "forward_consume":
        return {"send": pooled, "recv": pooled, "flags": None}
    return {"send": pooled, "flags": None}
