"""Performance cases of the library: the calls its users make, over the sizes they make them at.

A case is one call of one public entry point of the Python binding, with the
inputs, outputs and workspace a program keeps between calls already on the
GPU.  The families follow the header: map, transform_reduce (sums and dot
products), the fused map + reduce, the grouped batch, segmented reduce, scan
and segmented scan.  Sizes run from 2^10 elements, where the launch counts, to
the 2^28 of the bandwidth workload; values are the uniform, normal and
lognormal ones of the repository's own workloads.

Keys of a case: op, dtype, acc, fn (fold callable), map_fn, n (elements; of
the whole range for segments, of the largest call for a batch), shift (the
inputs are views that start this many elements into their buffer), and per
family mean_len (segments), calls (batch), exclusive (scans).
"""
import torch

import paper_2309_03912_amd as hdc

DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "i32": torch.int32}
CODE = {"f32": hdc.F32, "f16": hdc.F16, "bf16": hdc.BF16, "i32": hdc.I32}
SIZE = {"f32": 4, "f16": 2, "bf16": 2, "i32": 4}
OUT_SIZE = {"plain": 4, "compensated": 8, "exact_int": 8, "exact": 8}
COEF = [1.0 / (k + 1) for k in range(9)]  # the degree-8 polynomial of the workloads
DEV = "cuda:0"
BATCH_SPREAD = 12  # the calls of a batch span 2^-12 .. 1 of its largest one


def case(name, op, dtype, acc, fn, n, **more):
    return {"name": name, "op": op, "dtype": dtype, "acc": acc, "fn": fn, "n": n, "shift": 0, **more}


def listed():
    return [
        # the smallest calls, in a loop of many: what a call costs by itself
        case("map_f32_small", "map", "f32", "plain", "affine", 4097),
        # the bandwidth workload's longest operation
        case("map_i32_large", "map", "i32", "exact_int", "affine", 1 << 28),
        # a slice of a larger buffer mapped into a buffer of its own: 16-bit storage, ragged, operands aligned apart
        case("map_bf16_slice", "map", "bf16", "plain", "horner", (1 << 25) + 13, shift=3),
        # the small workload: a sum over an array that fits the caches
        case("sum_f32_small", "reduce", "f32", "plain", "horner", 1 << 20),
        # the precision workload: a compensated dot product in 16-bit storage
        case("dot_bf16_large", "dot", "bf16", "compensated", "product", 1 << 28),
        # a bit-reproducible (exact) sum, odd size
        case("sum_bf16_exact", "reduce", "bf16", "exact", "identity", (1 << 27) + 5),
        # one call of the graph workload: fp16 map and compensated sum in one pass, ordinary size
        case("map_reduce_f16", "map_reduce", "f16", "compensated", "horner", 3_000_001, map_fn="affine"),
        # the graph workload's int32 calls as one grouped batch: many sizes in one call
        case("batch_i32", "batch", "i32", "exact_int", "identity", 1 << 24, map_fn="affine", calls=32),
        # the batching workload: 100,000 lognormal segments over 1.3e8 elements
        case("seg_f32_lognormal", "segmented", "f32", "plain", "horner", 134_000_000, mean_len=1340),
        # many short rows of an ordinary size (a sparse matrix, a ragged mini-batch), 16-bit storage
        case("seg_bf16_rows", "segmented", "bf16", "compensated", "identity", 2_000_003, mean_len=48),
        # exclusive prefix sums of counts (offsets of a compaction), odd size
        case("scan_i32_exclusive", "scan", "i32", "exact_int", "identity", (1 << 27) + 3, exclusive=True),
        # running sums that restart at every segment
        case("segscan_f32", "segscan", "f32", "plain", "horner", 134_000_000, mean_len=1340, exclusive=False),
    ]


def log_size(rng, lo, hi):
    """A size spread over its logarithm; two in three are odd or ragged."""
    n = int(2.0 ** rng.uniform(lo, hi))
    return n if rng.random() < 0.67 else max(1 << 10, n // 1024 * 1024)


def draw(rng):
    op = rng.choice(["map", "reduce", "dot", "map_reduce", "batch", "segmented", "scan", "segscan"])
    shift = rng.choice([0, 0, 0, 0, 1, 3])
    fold = [("f32", "plain", "horner"), ("f32", "compensated", "horner"), ("f16", "compensated", "horner"),
            ("bf16", "compensated", "identity"), ("i32", "exact_int", "identity"), ("i32", "exact_int", "affine")]
    if op == "map":
        dtype, fn = rng.choice([("f32", "affine"), ("f32", "horner"), ("f16", "affine"), ("bf16", "horner"),
                                ("i32", "affine")])
        c = {"acc": "exact_int" if dtype == "i32" else "plain", "fn": fn, "n": log_size(rng, 10, 28)}
    elif op == "reduce":
        dtype, acc, fn = rng.choice(fold + [("f16", "exact", "identity"), ("bf16", "exact", "identity")])
        c = {"acc": acc, "fn": fn, "n": log_size(rng, 10, 28)}
    elif op == "dot":
        dtype, acc = rng.choice([("f32", "plain"), ("bf16", "compensated"), ("f16", "compensated"), ("f16", "exact")])
        c = {"acc": acc, "fn": "product", "n": log_size(rng, 10, 27 if dtype == "f32" else 28)}
    elif op == "map_reduce":
        dtype, acc, fn = rng.choice(fold)
        c = {"acc": acc, "fn": fn, "n": log_size(rng, 10, 27), "map_fn": "affine"}
    elif op == "batch":
        dtype, acc, fn = rng.choice([("f32", "plain", "horner"), ("f16", "compensated", "horner"),
                                     ("i32", "exact_int", "identity")])
        c = {"acc": acc, "fn": fn, "n": log_size(rng, 12, 24), "map_fn": "affine", "calls": rng.randint(2, 32)}
    elif op == "segmented":
        dtype, acc, fn = rng.choice(fold)
        c = {"acc": acc, "fn": fn, "n": log_size(rng, 14, 27), "mean_len": int(2.0 ** rng.uniform(4, 13))}
    else:
        dtype, acc, fn = rng.choice(fold)
        c = {"acc": acc, "fn": fn, "n": log_size(rng, 11, 27), "exclusive": rng.random() < 0.4}
        if op == "segscan":
            c["mean_len"] = int(2.0 ** rng.uniform(4, 13))
    return {"op": op, "dtype": dtype, "shift": shift, **c}


# --- inputs ------------------------------------------------------------------

def generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def values(g, c, n):
    """n values of the case's storage: counts below 2^20 (int32), U[-1, 1) under a polynomial, N(0, 1) otherwise."""
    buf = torch.empty(n + c["shift"], dtype=DTYPE[c["dtype"]], device=DEV)
    if c["dtype"] == "i32":
        buf.random_(0, 1 << 20, generator=g)
    elif c["fn"] == "horner" or c["op"] == "map":
        buf.uniform_(-1.0, 1.0, generator=g)
    else:
        buf.normal_(0.0, 1.0, generator=g)
    return buf[c["shift"]:]


def segment_offsets(g, c):
    """CSR offsets of lognormal segment lengths that cover the n elements, mean_len on average; some are empty."""
    sigma = 1.8  # the workload's spread: median 256 for a mean of 1342
    count = max(1, c["n"] // c["mean_len"])
    length = torch.exp(sigma * torch.randn(count, generator=g, device=DEV, dtype=torch.float64))
    ends = (torch.cumsum(length, 0) * (c["n"] / length.sum())).to(torch.int64).clamp_(max=c["n"])
    ends[-1] = c["n"]
    return torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), ends])


def batch_sizes(c):
    """Sizes of a batch's calls, spread over their logarithm up to n (the same for every seed, as in the workload)."""
    k = c["calls"]
    return [max(1 << 10, int(c["n"] * 2.0 ** (-BATCH_SPREAD * ((5 * i) % k) / k)) | (i & 1)) for i in range(k)]


def callable_of(c, fn):
    if fn == "affine":
        return hdc.affine(3, -7) if c["dtype"] == "i32" else hdc.affine(2.5, 0.5)
    return {"identity": hdc.identity, "product": hdc.product}[fn]() if fn != "horner" else hdc.horner(COEF)


def inputs(c, seed):
    g = generator(seed)
    if c["op"] == "batch":
        return {"xs": [values(g, c, n) for n in batch_sizes(c)]}
    s = {"x": values(g, c, c["n"])}
    if c["op"] == "dot":  # correlated operands, as in a projection
        z = torch.empty(c["n"] + c["shift"], dtype=DTYPE[c["dtype"]], device=DEV).normal_(0.0, 1.0, generator=g)
        z = z[c["shift"]:]
        s["z"] = z.add_(s["x"], alpha=0.5)
    if c["op"] in ("segmented", "segscan"):
        s["offsets"] = segment_offsets(g, c)
    return s


def prepare(c, seed):
    """The inputs, the callables, and the outputs and workspace that a program keeps between calls."""
    s = dict(inputs(c, seed), case=c, fn=callable_of(c, c["fn"]))
    if "map_fn" in c:
        s["map_fn"] = callable_of(c, c["map_fn"])
    acc = hdc.ACC[c["acc"]]
    scalar = lambda: torch.empty((), dtype=hdc.OUT_DTYPE[acc], device=DEV)  # noqa: E731
    op = {"map": hdc.OP_MAP, "reduce": hdc.OP_TRANSFORM_REDUCE, "dot": hdc.OP_TRANSFORM_REDUCE,
          "map_reduce": hdc.OP_MAP_REDUCE, "batch": hdc.OP_BATCH, "segmented": hdc.OP_SEGMENTED_REDUCE,
          "scan": hdc.OP_SCAN, "segscan": hdc.OP_SCAN}[c["op"]]
    total, count = c["n"], 0
    if c["op"] == "map":
        s["y"] = torch.empty(c["n"], dtype=DTYPE[c["dtype"]], device=DEV)
    elif c["op"] in ("reduce", "dot"):
        s["out"] = scalar()
    elif c["op"] == "map_reduce":
        s["y"] = torch.empty(c["n"], dtype=DTYPE[c["dtype"]], device=DEV)
        s["out"] = scalar()
    elif c["op"] == "batch":
        s["ys"] = [torch.empty_like(x) for x in s["xs"]]
        s["outs"] = [scalar() for _ in s["xs"]]
        total, count = sum(x.numel() for x in s["xs"]), len(s["xs"])
    elif c["op"] == "segmented":
        count = s["offsets"].numel() - 1
        s["out"] = torch.empty(count, dtype=hdc.OUT_DTYPE[acc], device=DEV)
    else:
        s["y"] = torch.zeros(c["n"], dtype=hdc.OUT_DTYPE[acc], device=DEV)
    if c["op"] != "map":
        need = hdc.workspace_size(op, CODE[c["dtype"]], acc, total, count)
        s["ws"] = torch.zeros(max(need, 256), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    """One call."""
    c = s["case"]
    op, acc = c["op"], c["acc"]
    if op == "map":
        return hdc.map(s["x"], s["fn"], out=s["y"])
    if op == "reduce":
        return hdc.transform_reduce(s["x"], s["fn"], acc, out=s["out"], ws=s["ws"])
    if op == "dot":
        return hdc.transform_reduce(s["x"], s["fn"], acc, z=s["z"], out=s["out"], ws=s["ws"])
    if op == "map_reduce":
        return hdc.map_reduce(s["x"], s["map_fn"], s["fn"], acc, out=s["y"], result=s["out"], ws=s["ws"])
    if op == "batch":
        return hdc.batch_map_reduce(s["xs"], s["map_fn"], s["fn"], acc, ys=s["ys"], outs=s["outs"], ws=s["ws"])
    if op == "segmented":
        return hdc.segmented_reduce(s["x"], s["offsets"], s["fn"], acc, out=s["out"], ws=s["ws"])
    if op == "scan":  # asynchronous, as inside a stream of work
        return hdc.scan(s["x"], s["fn"], acc, c["exclusive"], out=s["y"], ws=s["ws"], check=False)
    return hdc.segmented_scan(s["x"], s["offsets"], s["fn"], acc, c["exclusive"], out=s["y"], ws=s["ws"], check=False)


def work(c):
    """Each input read once, each output written once; one multiply-add per polynomial step, one add per fold."""
    op, n, es = c["op"], c["n"], SIZE[c["dtype"]]
    per_term = {"identity": 0, "affine": 2, "horner": 2 * (len(COEF) - 1), "product": 1}
    if op == "map":
        return {"bytes": 2 * n * es, "flops": n * per_term[c["fn"]]}
    fold = per_term[c["fn"]] + 1
    if op == "reduce":
        return {"bytes": n * es, "flops": n * fold}
    if op == "dot":
        return {"bytes": 2 * n * es, "flops": n * fold}
    if op in ("map_reduce", "batch"):
        n = n if op == "map_reduce" else sum(batch_sizes(c))
        return {"bytes": 2 * n * es, "flops": n * (fold + per_term[c["map_fn"]])}
    segments = max(1, n // c["mean_len"]) if "mean_len" in c else 0
    if op == "segmented":
        return {"bytes": n * es + segments * (8 + OUT_SIZE[c["acc"]]), "flops": n * fold}
    return {"bytes": n * (es + OUT_SIZE[c["acc"]]) + 8 * segments, "flops": n * fold}


# --- the same in 64 bits, in plain torch ---------------------------------------

def apply64(c, fn, x):
    x = x.double()
    if fn == "affine":
        return x.mul_(2.5).add_(0.5)
    if fn == "horner":
        coef = torch.tensor(COEF, dtype=torch.float32).double().tolist()  # the callable's coefficients are fp32
        acc = torch.full_like(x, coef[-1])
        for a in reversed(coef[:-1]):
            acc.mul_(x).add_(a)
        return acc
    return x


def exact(c, seed):
    """The outputs of run() in fp64; None for integers, which are compared bit by bit."""
    if c["dtype"] == "i32":
        return None
    s = inputs(c, seed)
    op = c["op"]
    if op == "map":
        return apply64(c, c["fn"], s["x"])
    if op == "dot":
        step = 1 << 26
        return sum((a.double() * b.double()).sum() for a, b in zip(s["x"].split(step), s["z"].split(step)))
    if op == "batch":
        return ([apply64(c, c["map_fn"], x) for x in s["xs"]], [apply64(c, c["fn"], x).sum() for x in s["xs"]])
    if op == "map_reduce":
        return apply64(c, c["map_fn"], s["x"]), apply64(c, c["fn"], s["x"]).sum()
    if op == "reduce":
        return sum(apply64(c, c["fn"], x).sum() for x in s["x"].split(1 << 26))
    t = apply64(c, c["fn"], s["x"])
    if op == "segmented":
        return torch.segment_reduce(t, "sum", offsets=s["offsets"], initial=0.0)
    y = torch.cumsum(t, 0)
    before = y - t  # the exclusive prefix
    if op == "segscan":
        length = s["offsets"][1:] - s["offsets"][:-1]
        start = s["offsets"][:-1].clamp(max=c["n"] - 1)
        base = torch.repeat_interleave(before[start], length, output_size=c["n"])
        y, before = y - base, before - base
    return before if c["exclusive"] else y
