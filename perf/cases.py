"""What is timed of the cached embedding-bag training path, and how its results are checked.

A pass is a few training steps of one model through the public calls, as a training loop makes them: prefetch of
the next batch, pooled forward of the current one, backward with the fused row-wise Adagrad update, and where a case
says so a flush at the end (a checkpoint).  A state's batches follow one another from pass to pass like a stream, and
every pass of more steps than there are batches looks some rows up again that it has updated, so that the pooled
vectors it returns depend on its own updates; a pass that flushes returns the updated tables and accumulators too.

Fields of a case:
  tables, rows, dim   tables of `rows` rows of `dim` elements; with `mixed` the tables differ: rows spread over their
                      logarithm up to `rows`, 64, 128 or 256 elements, mean pooling lengths up to `pool`, Zipf 0.9-1.3
  half                rows stored as binary16 (else fp32)
  batch, pool, fixed  samples per batch, lookups per bag: `fixed` or Poisson, at least `pool_min`, at most 200
  alpha, reuse        Zipf exponent of the row popularity (0: uniform), share of the lookups that repeat the batch before
  ways, cache         associativity, cached share of the rows
  ahead, depth        batches prefetched ahead by the loop (0: none), depth of the library's pipeline
  batches, steps      distinct batches of the stream, steps of a pass
  warm                steps trained before the first pass
  policy, pooling, level2, flush   options of the library, see include/tbe.h
"""
import math

import numpy as np
import torch

LR, EPS, INIT_STD = 0.01, 1e-8, 0.01

_BASE = {"mixed": False, "half": True, "fixed": False, "pool_min": 0, "reuse": 0.0, "ahead": 1, "depth": 1, "warm": 0,
         "policy": "lru", "pooling": "sum", "level2": 0, "flush": False}


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # The smallest calls: a unit test, a first look at a model, the last ragged batch of an epoch.  No loop that
        # prefetches ahead; what counts is the latency of a call.
        _case("smallest", tables=2, rows=2000, dim=16, half=False, batch=16, pool=4.0, alpha=1.05, ways=8, cache=0.25,
              ahead=0, batches=3, steps=2),
        # The small configuration of this repository (4 x 100k x 64 fp32, batch 512): small models, small batches.
        _case("tiny", tables=4, rows=100_000, dim=64, half=False, batch=512, pool=20.0, fixed=True, alpha=1.05, ways=32,
              cache=0.10, batches=5, steps=6),
        # The same model with a checkpoint after every other step: flush, host tables and accumulators current.
        _case("tiny_checkpoint", tables=4, rows=100_000, dim=64, half=False, batch=512, pool=20.0, fixed=True, alpha=1.05,
              ways=32, cache=0.10, batches=3, steps=2, flush=True),
        # The benchmark: 32 x 1M x 128 fp16, batch 8192, Zipf 1.1, 5 % cached, next batch prefetched ahead.
        _case("main", tables=32, rows=1_000_000, dim=128, batch=8192, pool=30.0, pool_min=1, alpha=1.1, ways=64, cache=0.05,
              batches=3, steps=4),
        # A model that fits the cache: every row hits after the first epoch, the host link is idle (shapes of the
        # benchmark with half its tables).
        _case("resident", tables=16, rows=500_000, dim=128, batch=8192, pool=30.0, pool_min=1, alpha=1.1, ways=64, cache=1.0,
              batches=2, steps=4, warm=2),
        # Capacity-bound: few large tables, large batches, short-term reuse (8 tables, 1/16 of the configuration's rows).
        _case("capacity", tables=8, rows=4_000_000, dim=128, batch=32768, pool=40.0, pool_min=1, alpha=1.05, reuse=0.3,
              ways=64, cache=1 / 16, batches=3, steps=4),
        # Heterogeneous: many tables of unlike size, width, pooling and skew.
        _case("hetero", tables=60, rows=1_000_000, dim=0, mixed=True, batch=4096, pool=100.0, alpha=0.0, ways=64, cache=0.08,
              batches=3, steps=4),
        # One point of the locality sweep: one large table of 64 elements, a tenth of its rows.
        _case("locality", tables=1, rows=10_000_000, dim=64, batch=32768, pool=32.0, fixed=True, alpha=1.0, ways=64,
              cache=0.05, batches=4, steps=5),
        # Mean pooling of fp32 rows of an odd width, ragged bags, many of them empty or short, an odd batch.
        _case("mean_ragged", tables=10, rows=200_000, dim=100, half=False, batch=3001, pool=3.0, alpha=0.8, ways=16,
              cache=0.10, pooling="mean", batches=3, steps=4),
        # Max pooling.
        _case("max", tables=8, rows=500_000, dim=128, batch=4096, pool=25.0, alpha=1.1, ways=64, cache=0.20, pooling="max",
              batches=2, steps=3),
        # Pipeline two batches deep with LFU replacement, uniform-ish accesses.
        _case("deep_lfu", tables=4, rows=1_000_000, dim=64, batch=4096, pool=16.0, alpha=0.9, ways=32, cache=0.25, ahead=2,
              depth=2, policy="lfu", batches=4, steps=5),
        # Two cache levels.
        _case("two_level", tables=4, rows=500_000, dim=128, batch=4096, pool=20.0, alpha=1.05, ways=32, cache=0.05, level2=2,
              batches=4, steps=5),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """Any model of the listed ranges: 1 to 32 tables, widths of every kind the library takes, bags from none to 60
    lookups, batches of 1 to 16384 samples, every option."""
    c = dict(_BASE)
    c["half"] = rng.random() < 0.6
    c["mixed"] = rng.random() < 0.15
    c["tables"] = int(_log(rng, 8, 60)) if c["mixed"] else int(_log(rng, 1, 33))
    c["dim"] = 0 if c["mixed"] else (8 if c["half"] else 4) * rng.choice([1, 2, 3, 4, 5, 8, 8, 12, 16, 16, 25, 32])
    width = 256 if c["mixed"] else c["dim"]
    row_bytes = width * (2 if c["half"] else 4)
    c["rows"] = int(_log(rng, 1e3, min(2e6, 2e9 / (c["tables"] * row_bytes))))
    if c["mixed"]:
        c["rows"] = max(20_000, c["rows"])
    c["alpha"] = rng.choice([0.0, round(rng.uniform(0.7, 1.4), 3), round(rng.uniform(0.9, 1.2), 3)])
    c["pool"] = round(_log(rng, 1.0, 60.0), 2)
    c["fixed"] = rng.random() < 0.3
    if c["fixed"]:
        c["pool"] = float(max(1, int(c["pool"])))
    c["pool_min"] = 0 if c["fixed"] else rng.choice([0, 1])
    most = min(4e6, 1e9 / row_bytes) / (c["tables"] * max(1.0, c["pool"]))
    c["batch"] = int(_log(rng, 1, max(2.0, min(16385.0, most))))
    if c["batch"] < 16:
        c["pool_min"] = 1
    c["ways"] = rng.choice([4, 8, 16, 32, 64, 64])
    c["cache"] = rng.choice([round(_log(rng, 0.02, 0.5), 4), round(_log(rng, 0.02, 0.5), 4), 1.0])
    c["pooling"] = rng.choice(["sum", "sum", "sum", "mean", "max"])
    c["policy"] = rng.choice(["lru", "lru", "lfu"])
    c["ahead"] = rng.choice([0, 1, 1, 1, 2])
    c["depth"] = max(1, c["ahead"])
    if c["depth"] == 1 and rng.random() < 0.2 and c["rows"] * c["cache"] >= c["ways"]:
        c["level2"] = rng.choice([1, 2])
    c["reuse"] = rng.choice([0.0, 0.0, 0.3])
    c["batches"], c["steps"] = rng.choice([2, 3]), rng.choice([2, 3]) if c["pooling"] == "max" else rng.choice([2, 3, 4])
    c["flush"] = not c["mixed"] and c["tables"] * c["rows"] * row_bytes < 5e7 and rng.random() < 0.5
    return c


# ---- the model a case describes ----

def _tables(case):
    """(rows, dim, Zipf exponent, mean bag length, cache slots) of every table: a function of the case alone."""
    out = []
    for t in range(case["tables"]):
        rows, dim, alpha, pool = case["rows"], case["dim"], case["alpha"], case["pool"]
        if case["mixed"]:
            u = np.random.RandomState(977 + t).rand(4)
            rows = int(round(10_000 * (case["rows"] / 10_000) ** u[0]))
            dim = (64, 128, 256)[int(u[1] * 3)]
            pool = case["pool"] ** u[2]
            alpha = 0.9 + 0.4 * u[3]
        slots = rows + case["ways"] if case["cache"] >= 1.0 else int(rows * case["cache"])
        out.append((rows, dim, alpha, pool, slots))
    return out


def _gen(seed, *stream):
    s = seed & 0xFFFFFFFF
    for x in stream:
        s = (s * 1000003 + (x + 1) * 7919 + 12345) % ((1 << 61) - 1)
    return torch.Generator(device="cuda").manual_seed(s)


def _weights(case, seed, t, rows, dim):
    w = torch.randn(rows, dim, generator=_gen(seed, 1, t), device="cuda") * INIT_STD
    return w.half() if case["half"] else w


def _batches(case, seed):
    """The stream's distinct batches: (indices of every table's bags one behind the other, offsets)."""
    tabs, B = _tables(case), case["batch"]
    got, before = [], None
    for k in range(case["batches"]):
        idx, lens = [], []
        for t, (rows, _, alpha, pool, _) in enumerate(tabs):
            g = _gen(seed, 2, t, k)
            if case["fixed"]:
                n = torch.full((B,), int(pool), dtype=torch.int64, device="cuda")
            else:
                n = torch.poisson(torch.full((B,), float(pool), dtype=torch.float64, device="cuda"), generator=g)
                n = n.to(torch.int64).clamp_(case["pool_min"], 200)
            total = int(n.sum())
            u = torch.rand(total, generator=g, dtype=torch.float64, device="cuda")
            if alpha == 0.0:
                r = torch.floor(u * rows)
            elif abs(alpha - 1.0) < 1e-12:
                r = torch.floor(torch.exp(u * math.log(rows + 1.0))) - 1.0
            else:
                r = torch.floor((((rows + 1.0) ** (1.0 - alpha) - 1.0) * u + 1.0) ** (1.0 / (1.0 - alpha))) - 1.0
            r = r.clamp_(0, rows - 1).to(torch.int64)
            a = int(rows * 0.6180339887) + t  # popularity rank -> row: an affine map that is one to one
            a = max(1, a)
            while math.gcd(a, rows) != 1:
                a += 1
            r = (r * a + (seed * 31 + t * 7) % rows) % rows
            if before is not None and case["reuse"] > 0 and total and before[t].numel():
                take = torch.rand(total, generator=g, device="cuda") < case["reuse"]
                pick = torch.randint(0, before[t].numel(), (total,), generator=g, device="cuda")
                r = torch.where(take, before[t][pick], r)
            idx.append(r)
            lens.append(n)
        before = idx
        off = torch.zeros(len(tabs) * B + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(torch.cat(lens), 0, out=off[1:])
        got.append((torch.cat(idx).contiguous(), off))
    return got


def _grads(case, seed):
    width = sum(t[1] for t in _tables(case))
    return [torch.randn(case["batch"], width, generator=_gen(seed, 3, k), device="cuda") for k in range(2)]


# ---- a user's program ----

class _State:
    pass


_pinned_for = None


def prepare(case, seed):
    from paper_2305_01515_amd.tbe import TBE, pinned_empty
    global _pinned_for
    shape = tuple(t[:2] for t in _tables(case)) + (case["half"],)
    if shape != _pinned_for:  # pinned blocks of another model's size are of no use and count against the machine's limit
        torch.cuda.synchronize()
        torch._C._host_emptyCache()
        _pinned_for = shape
    s = _State()
    s.case, s.batches, s.grads, s.at = case, _batches(case, seed), _grads(case, seed), 0
    s.weights, s.state = [], []
    for t, (rows, dim, _, _, _) in enumerate(_tables(case)):
        w = pinned_empty((rows, dim), torch.float16 if case["half"] else torch.float32)
        w.copy_(_weights(case, seed, t, rows, dim))
        s.weights.append(w)
        s.state.append(pinned_empty((rows,), torch.float32).zero_())
    most = max(1, max(b[0].numel() for b in s.batches))
    s.tbe = TBE(s.weights, s.state, [t[4] for t in _tables(case)], case["ways"], case["batch"], most, policy=case["policy"],
                pooling=case["pooling"], second_level_factor=case["level2"])
    if case["depth"] > 1:
        s.tbe.set_prefetch_depth(case["depth"])
    torch.cuda.synchronize()
    if case["ahead"]:
        s.tbe.set_inputs_ready(True)  # the batches were complete before the loop began
    if case["warm"]:
        _train(s, case["warm"])
        torch.cuda.synchronize()
    return s


def _train(s, steps):
    ahead, outs = s.case["ahead"], []
    order = [s.at + i for i in range(steps)]
    batch = lambda i: s.batches[i % len(s.batches)]  # noqa: E731
    for i in order[:ahead]:
        s.tbe.prefetch(*batch(i))
    for n, i in enumerate(order):
        if ahead and n + ahead < steps:
            s.tbe.prefetch(*batch(order[n + ahead]))
        outs.append(s.tbe.forward(*batch(i)))
        s.tbe.backward_update(s.grads[i % len(s.grads)], LR, EPS)
    s.at += steps
    return outs


def run(s):
    out = {"pooled": _train(s, s.case["steps"])}
    if s.case["flush"]:
        s.tbe.flush()
        out["weights"], out["state"] = s.weights, s.state
    return out


# ---- what a pass cannot do without ----

def _distinct(n, rows, alpha):
    """Expected number of distinct rows among n lookups."""
    if alpha == 0.0:
        return rows * -math.expm1(n * math.log1p(-1.0 / rows)) if rows > 1 else 1.0
    head = min(rows, 4096)
    edges = np.arange(1, head + 2, dtype=np.float64)
    if rows > head:
        edges = np.concatenate([edges, np.exp(np.linspace(math.log(head + 1.0), math.log(rows + 1.0), 4000))[1:]])
    cdf = np.log(edges) / math.log(rows + 1.0) if abs(alpha - 1.0) < 1e-12 else (edges ** (1 - alpha) - 1) / ((rows + 1.0) ** (1 - alpha) - 1)
    ranks = np.diff(edges)
    return float(np.sum(ranks * -np.expm1(-n * np.diff(cdf) / ranks)))


def work(case):
    """Per step: indices and offsets, the output gradient and the pooled vectors once, every distinct row and its
    accumulator read once and written once; a flush writes the cached rows and all accumulators."""
    B, per_step, flops, flush = case["batch"], 0.0, 0.0, 0.0
    for rows, dim, alpha, pool, slots in _tables(case):
        row = dim * (2 if case["half"] else 4)
        n = B * pool
        per_step += 8 * n + 8 * B + 8 * B * dim + _distinct(n, rows, alpha) * 2 * (row + 4)
        flops += 2 * n * dim + 5 * _distinct(n, rows, alpha) * dim
        flush += min(rows, slots) * row + 4 * rows
    return {"bytes": case["steps"] * per_step + (flush if case["flush"] else 0.0), "flops": case["steps"] * flops}


def tolerance(case):
    """fp32 sums of up to thousands of terms in another order differ by some 1e-7.  Where such a difference tips the
    rounding of a stored binary16 row (about one update in 5000), the element is one unit off from then on: 4e-6 to 1e-5
    in the 2-norm.  Under max pooling it now and then decides between two rows of almost one value, and the gradient
    goes to the other one: single elements are then quite different."""
    if case["pooling"] == "max":
        return {"rel": 1e-2 if case["half"] else 1e-3, "max": 0.99}
    return {"rel": 5e-5, "max": 4e-3} if case["half"] else {"rel": 2e-6, "max": 1e-4}


# ---- the same in 64 bits ----

def exact(case, seed):
    tabs, B = _tables(case), case["batch"]
    batches, grads = _batches(case, seed), _grads(case, seed)
    order = [i % len(batches) for i in range(case["warm"] + case["steps"])]
    pooled = [torch.empty(B, sum(t[1] for t in tabs), dtype=torch.float64, device="cuda") for _ in range(case["steps"])]
    out_w, out_m, col = [], [], 0
    for t, (rows, dim, _, _, _) in enumerate(tabs):
        W = _weights(case, seed, t, rows, dim)
        part = []  # (row of the touched ones, bag, bag lengths) of every batch
        for idx, off in batches:
            o = off[t * B:(t + 1) * B + 1]
            part.append((idx[int(o[0]):int(o[-1])], o[1:] - o[:-1]))
        touched, where = torch.unique(torch.cat([p[0] for p in part]), return_inverse=True)
        where = torch.split(where, [p[0].numel() for p in part])
        w = W[touched].double()
        m = torch.zeros(touched.numel(), dtype=torch.float64, device="cuda")
        for n, i in enumerate(order):
            u, lens = where[i], part[i][1]
            bag = torch.repeat_interleave(torch.arange(B, device="cuda"), lens)
            g = grads[n % len(grads)][:, col:col + dim].double()
            scale = 1.0 / lens.clamp(min=1).double() if case["pooling"] == "mean" else None
            if case["pooling"] == "max":
                at = bag[:, None].expand(-1, dim)
                best = torch.full((B, dim), -math.inf, dtype=torch.float64, device="cuda").scatter_reduce_(0, at, w[u], "amax")
                place = torch.arange(u.numel(), device="cuda")[:, None].expand(-1, dim)
                none = u.numel()
                first = torch.full((B, dim), none, dtype=torch.int64, device="cuda")
                first.scatter_reduce_(0, at, torch.where(w[u] == best[bag], place, none), "amin")
                p = torch.where(lens[:, None] > 0, best, 0.0)
                per_lookup = torch.where(first[bag] == place, g[bag], 0.0)
            else:
                p = torch.zeros(B, dim, dtype=torch.float64, device="cuda").index_add_(0, bag, w[u])
                if scale is not None:
                    p *= scale[:, None]
                    g = g * scale[:, None]
                per_lookup = g[bag]
            if n >= case["warm"]:
                pooled[n - case["warm"]][:, col:col + dim] = p
            G = torch.zeros_like(w).index_add_(0, u, per_lookup)
            del per_lookup
            hit = torch.zeros(touched.numel(), dtype=torch.bool, device="cuda")
            hit[u] = True
            m = torch.where(hit, m + G.square().mean(1), m)
            w = torch.where(hit[:, None], w - LR * G / (m.sqrt() + EPS)[:, None], w)
        if case["flush"]:
            full = W.double()
            full[touched] = w
            acc = torch.zeros(rows, dtype=torch.float64, device="cuda")
            acc[touched] = m
            out_w.append(full.cpu())
            out_m.append(acc.cpu())
        col += dim
    out = {"pooled": pooled}
    if case["flush"]:
        out["weights"], out["state"] = out_w, out_m
    return out
