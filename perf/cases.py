"""The work that programs have this library do, as cases that can be timed.

Three operations, each through the call that a program makes (the library
and the plan cache are loaded once, at import, as the README's example does;
calls run on the current stream):

* ``sum``       -- ``redsum.sum(x)``, compensated accumulation (the default;
                   it costs no more than plain accumulation);
* ``segments``  -- ``redsum.segmented_sum(values, offsets)``;
* ``stencil``   -- ``redsum.jacobi(u, steps, r)``, in place.

``prepare`` draws everything on the GPU from the seed.  Values are N(0, 1)
(int32: uniform on [-1000, 1000]); an array may start ``shift`` elements into
its allocation, as a view does.
"""
import math

import torch

from paper_2004_05371_amd import autotune, redsum

redsum.load()
autotune.load()

DTYPES = {"f32": torch.float32, "i32": torch.int32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZES = {"f32": 4, "i32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # A metric or a loss term over one small array: latency alone.
        {"name": "sum_f32_1000", "op": "sum", "dtype": "f32", "n": 1000, "shift": 0},
        # A layer's bias or activation row, odd length.
        {"name": "sum_bf16_100003", "op": "sum", "dtype": "bf16", "n": 100003, "shift": 0},
        # The small workload of the benchmark.
        {"name": "sum_i32_2p20", "op": "sum", "dtype": "i32", "n": 1 << 20, "shift": 0},
        # An ordinary array in the caches, of odd size and not aligned to 16 bytes.
        {"name": "sum_f16_5m", "op": "sum", "dtype": "f16", "n": 5000011, "shift": 3},
        # The headline workload of the benchmark: 1 GiB from HBM.
        {"name": "sum_f32_2p28", "op": "sum", "dtype": "f32", "n": 1 << 28, "shift": 0},
        # A small batch of rows, as one request of a service brings.
        {"name": "seg_small", "op": "segments", "nseg": 300, "total": 60000, "dist": "geometric", "shift": 0},
        # Rows of a sparse matrix or neighbours of a graph's nodes: short, uneven, some empty.
        {"name": "seg_short", "op": "segments", "nseg": 2000003, "total": 32000000, "dist": "geometric", "shift": 0},
        # Fixed-length rows (feature vectors, tokens of equal sequences).
        {"name": "seg_rows_512", "op": "segments", "nseg": 131072, "total": 131072 * 512, "dist": "equal", "shift": 0},
        # The segmented workload of the benchmark: 10,000 log-uniform lengths up to about 2^20.
        {"name": "seg_drawn", "op": "segments", "nseg": 10000, "total": 742706513, "dist": "loguniform", "shift": 0},
        # A small grid stepped many times (the stencil's smallest size in the benchmark).
        {"name": "stencil_64k", "op": "stencil", "n": 65536, "steps": 1000, "r": 0.25},
        # The stencil workload of the benchmark's line.
        {"name": "stencil_4m", "op": "stencil", "n": 4194304, "steps": 200, "r": 0.25},
        # A grid that the chip's registers do not hold.
        {"name": "stencil_24m", "op": "stencil", "n": 24000001, "steps": 40, "r": 0.3},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["sum", "sum", "segments", "segments", "stencil"])
    if op == "sum":
        dtype = rng.choice(["f32", "f32", "i32", "f16", "bf16"])
        n = _log_int(rng, 256, (1 << 30) // SIZES[dtype])
        return {"op": op, "dtype": dtype, "n": n, "shift": rng.choice([0, 0, 1, 5])}
    if op == "segments":
        # 10^4 to 3 * 10^8 values in segments of 4 to 10^5 values on average.
        total = _log_int(rng, 10000, 300000000)
        mean = _log_int(rng, 4, 100000)
        nseg = max(1, total // mean)
        return {"op": op, "nseg": nseg, "total": total, "dist": rng.choice(["geometric", "equal", "loguniform"]),
                "shift": rng.choice([0, 0, 1])}
    n = _log_int(rng, 1000, 24000000)
    steps = min(_log_int(rng, 8, 1000), max(8, 900000000 // n))
    return {"op": op, "n": n, "steps": steps, "r": rng.choice([0.1, 0.25, 0.3, 0.5])}


def _values(case, gen, n):
    """n values of the case's type that start `shift` elements into an allocation."""
    shift = case.get("shift", 0)
    kind = case.get("dtype", "f32")
    if kind == "i32":
        x = torch.randint(-1000, 1001, (n + shift,), generator=gen, device="cuda", dtype=torch.int32)
    else:
        x = torch.randn(n + shift, generator=gen, device="cuda", dtype=torch.float32).to(DTYPES[kind])
    return x[shift:]


def _offsets(case, gen):
    """CSR offsets of `nseg` segments that hold `total` values together."""
    nseg, total, dist = case["nseg"], case["total"], case["dist"]
    off = torch.zeros(nseg + 1, dtype=torch.int64, device="cuda")
    if dist == "geometric":  # independent cuts: lengths from 0 up, their spread as large as their mean
        cuts = (torch.rand(nseg - 1, generator=gen, device="cuda", dtype=torch.float64) * (total + 1)).long()
        off[1:nseg] = torch.sort(cuts).values
    elif dist == "equal":  # equal lengths, the remainder spread over the segments
        k = torch.arange(1, nseg, device="cuda", dtype=torch.int64)
        off[1:nseg] = (k * (total // nseg)) + (k * (total % nseg)) // nseg
    else:  # log-uniform over the benchmark's 20 octaves, scaled to the total
        w = torch.exp(torch.rand(nseg, generator=gen, device="cuda", dtype=torch.float64) * math.log(1 << 20))
        off[1:nseg] = (torch.cumsum(w, 0)[:-1] * (total / w.sum())).long().clamp_(0, total)
    off[nseg] = total
    return off


def _make(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "sum":
        return {"x": _values(case, gen, case["n"])}
    if case["op"] == "segments":
        return {"offsets": _offsets(case, gen), "values": _values(case, gen, case["total"])}
    return {"u": _values(case, gen, case["n"]), "steps": case["steps"], "r": case["r"]}


def prepare(case, seed):
    return dict(_make(case, seed), op=case["op"])


def run(state):
    if state["op"] == "sum":
        return redsum.sum(state["x"])
    if state["op"] == "segments":
        return redsum.segmented_sum(state["values"], state["offsets"])
    return redsum.jacobi(state["u"], state["steps"], state["r"])


def exact(case, seed):
    s = _make(case, seed)
    if case["op"] == "sum":
        x = s["x"]
        return x.sum(dtype=torch.int64) if case["dtype"] == "i32" else x.double().sum()
    if case["op"] == "segments":
        off = s["offsets"]
        sums = torch.zeros(case["total"] + 1, dtype=torch.float64, device="cuda")
        torch.cumsum(s["values"], 0, dtype=torch.float64, out=sums[1:])
        return sums[off[1:]] - sums[off[:-1]]
    u, r = s["u"].double(), float(torch.tensor(case["r"], dtype=torch.float32))
    for _ in range(case["steps"]):
        v = u.clone()
        v[1:-1] += r * ((u[:-2] + u[2:]) - 2.0 * u[1:-1])
        u = v
    return u


def work(case):
    """Each input read once and each output written once; the additions (stencil: the step's five operations)."""
    if case["op"] == "sum":
        return {"bytes": case["n"] * SIZES[case["dtype"]] + 8, "flops": case["n"]}
    if case["op"] == "segments":
        return {"bytes": case["total"] * 4 + (case["nseg"] + 1) * 8 + case["nseg"] * 8, "flops": case["total"]}
    return {"bytes": case["n"] * 8, "flops": case["n"] * case["steps"] * 5.0}
