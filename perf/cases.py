"""Performance cases of the scan library: what its users have it do, through
the public entry points of ``paper_1604_04815_amd.binding``.

A case is a dict of plain values.  ``kind`` names the entry point:

* ``scan``       inclusive / exclusive plain scan (add, max, min, argmax,
                 argmin; optionally compensated, optionally of a slice)
* ``segmented``  one array cut by offsets
* ``batched``    many separate arrays in one launch
* ``compact``    stream compaction
* ``radix``      digit offsets of one radix-sort pass
* ``bfs``        breadth-first search

Inputs are drawn on the device from the seed alone, with the distributions
of the benchmark's workloads (``paper_1604_04815_amd/workloads.py``).  Every
state keeps its own output buffers, as a program that calls repeatedly does.
"""
from __future__ import annotations

import math

import torch

from paper_1604_04815_amd import binding, workloads

DEVICE = "cuda"
TORCH_DTYPE = {"int32": torch.int32, "int64": torch.int64, "float32": torch.float32, "bfloat16": torch.bfloat16}
IN_BYTES = {"int32": 4, "int64": 8, "float32": 4, "bfloat16": 2}


def _out_bytes(dtype: str, op: str = "add") -> int:
    return 8 if dtype == "int64" or op in ("argmax", "argmin") else 4


def _scan(name, n, dtype="int32", op="add", exclusive=False, compensated=False, offset=0):
    """offset: x starts this many elements into its buffer (a slice), y does not."""
    return {"name": name, "kind": "scan", "n": n, "dtype": dtype, "op": op, "exclusive": exclusive,
            "compensated": compensated, "offset": offset}


def listed():
    return [
        # the smallest calls: per-request sizes of the serving trace start at 2^10
        _scan("scan_i32_add_1k", 1000),
        # the latency workload of the benchmark
        _scan("scan_i32_add_1m", 1 << 20, exclusive=True),
        # the headline workload: a gigabyte-sized array, in one launch
        _scan("scan_i32_add_256m", 1 << 28),
        # long float sums where plain rounding is not good enough
        _scan("scan_f32_comp_128m", 1 << 27, "float32", compensated=True),
        # a 16-bit tensor's slice scanned into a fresh float32 output, odd length
        _scan("scan_bf16_add_slice", (1 << 26) + 5, "bfloat16", offset=3),
        # running arg-extremes of a long float series
        _scan("scan_f32_argmax_128m", (1 << 27) + 1, "float32", "argmax"),
        # 4096 arrays of very different lengths packed into one buffer
        {"name": "seg_f32_add_4096", "kind": "segmented", "n": 320_000_000, "segments": 4096, "dtype": "float32",
         "op": "add", "exclusive": False, "compensated": False},
        # ragged rows (compressed sparse rows, token lists): a million short segments
        {"name": "seg_i32_rows_1m", "kind": "segmented", "n": 25_000_003, "segments": 1 << 20, "dtype": "int32",
         "op": "add", "exclusive": True, "compensated": False},
        # the same 4096 arrays as separate requests batched into one launch
        {"name": "batch_i32_add_4096", "kind": "batched", "n": 320_000_000, "arrays": 4096, "dtype": "int32",
         "op": "add", "exclusive": False, "compensated": False},
        # filter a large column by a mask that keeps about half
        {"name": "compact_i32_256m", "kind": "compact", "n": 1 << 28, "dtype": "int32", "flags": True,
         "density": 0.5},
        # one 8-bit pass of a sort of 50 million keys
        {"name": "radix_i32_50m", "kind": "radix", "n": 50_000_017, "dtype": "int32", "shift": 8, "bits": 8,
         "block_items": 4096},
        # search of a scale-free graph, 4 million vertices and 134 million column entries
        {"name": "bfs_rmat22", "kind": "bfs", "scale": 22, "edge_factor": 16},
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["scan", "scan", "scan", "segmented", "batched", "compact", "radix", "bfs"])
    if kind == "bfs":
        return {"kind": kind, "scale": rng.randint(10, 21), "edge_factor": rng.randint(6, 16)}
    if kind == "radix":
        return {"kind": kind, "n": _log_uniform(rng, 1 << 12, 1 << 27), "dtype": rng.choice(["int32", "int64", "float32"]),
                "shift": rng.randint(0, 24), "bits": rng.randint(4, 8), "block_items": rng.choice([4096, 8192, 16384])}
    if kind == "compact":
        return {"kind": kind, "n": _log_uniform(rng, 1 << 10, 1 << 27), "dtype": rng.choice(["int32", "int64", "float32"]),
                "flags": rng.random() < 0.75, "density": round(rng.uniform(0.02, 0.98), 3)}
    dtype = rng.choice(["int32", "int64", "float32", "bfloat16"])
    op = rng.choice(["add", "add", "max", "min"])
    common = {"dtype": dtype, "op": op, "exclusive": rng.random() < 0.4,
              "compensated": dtype in ("float32", "bfloat16") and op == "add" and rng.random() < 0.4}
    if kind == "segmented":
        n = _log_uniform(rng, 1 << 12, 1 << 27)
        return {"kind": kind, "n": n, "segments": _log_uniform(rng, 1, max(2, n // 12)), **common}
    if kind == "batched":
        arrays = _log_uniform(rng, 8, 4096)
        return {"kind": kind, "n": _log_uniform(rng, arrays * 512, 1 << 27), "arrays": arrays, **common}
    if dtype != "bfloat16" and not common["compensated"] and rng.random() < 0.25:
        common["op"] = rng.choice(["argmax", "argmin"])
    return {"kind": kind, "n": _log_uniform(rng, 1 << 10, 1 << 27), "offset": rng.choice([0, 0, 0, 1, 2, 3]), **common}


def _generator(seed: int):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(workloads.BASE_SEED + int(seed))
    return g


def _values(dtype: str, op: str, n: int, g, positive=False):
    """n values on the device (the recipes of workloads.values_for)."""
    if dtype == "int32":
        lo, hi = (-1000, 1001) if op == "add" else (-(2 ** 31), 2 ** 31)
        return torch.randint(lo, hi, (n,), generator=g, device=DEVICE, dtype=torch.int32)
    if dtype == "int64":
        return torch.randint(-(2 ** 31), 2 ** 31, (n,), generator=g, device=DEVICE, dtype=torch.int64)
    if dtype == "bfloat16":
        return torch.rand(n, generator=g, device=DEVICE).to(torch.bfloat16)
    if positive:
        return torch.rand(n, generator=g, device=DEVICE)
    mag = torch.empty(n, device=DEVICE).log_normal_(0.0, 2.0, generator=g)
    return mag * (torch.randint(0, 2, (n,), generator=g, device=DEVICE) * 2 - 1)


def _offsets(n: int, parts: int, g):
    """parts + 1 offsets from 0 to n whose steps are log-uniform in [1, 2^20] up to one common factor."""
    w = torch.exp(torch.rand(parts, generator=g, device=DEVICE, dtype=torch.float64) * math.log(2 ** 20 if parts <= 65536 else 64))
    c = torch.cumsum(w, 0)
    off = torch.zeros(parts + 1, dtype=torch.int64, device=DEVICE)
    off[1:] = torch.round(c / c[-1] * n).to(torch.int64)
    off[-1] = n
    return off


def _graph(case, seed):
    row, col = workloads.rmat_csr_torch(case["scale"], case["edge_factor"], workloads.BASE_SEED + int(seed), device=DEVICE)
    deg = row[1:] - row[:-1]
    cand = torch.nonzero(deg > 0).flatten()
    return row, col, int(cand[(int(seed) * 2654435761) % cand.shape[0]].item())


def _inputs(case, seed):
    """The input tensors of a case other than a graph: (x, extra)."""
    g = _generator(seed)
    kind, n, dtype = case["kind"], case["n"], case["dtype"]
    if kind == "scan":
        off = case["offset"]
        return _values(dtype, case["op"], n + off, g)[off:], None
    if kind in ("segmented", "batched"):
        parts = case["segments"] if kind == "segmented" else case["arrays"]
        x = _values(dtype, case["op"], n, g, positive=True)
        return x, _offsets(n, parts, g)
    if kind == "compact":
        x = _values(dtype, "add", n, g)
        mask = torch.rand(n, generator=g, device=DEVICE) < case["density"]
        return (x, mask) if case["flags"] else (torch.where(mask, x, torch.zeros_like(x)), None)
    if dtype == "float32":
        return _values(dtype, "add", n, g), None
    return _values(dtype, "max", n, g), None


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "case": case}
    if kind == "bfs":
        s["row"], s["col"], s["source"] = _graph(case, seed)
        s["levels"] = torch.empty(s["row"].shape[0] - 1, dtype=torch.int32, device=DEVICE)
        s["stats"] = torch.empty(4, dtype=torch.int64, device=DEVICE)
        return s
    x, extra = _inputs(case, seed)
    s["x"], s["extra"] = x, extra
    n = case["n"]
    if kind == "compact":
        s["out"] = torch.zeros_like(x)  # only the kept items are written
        s["count"] = torch.zeros(1, dtype=torch.int64, device=DEVICE)
    elif kind == "radix":
        m = (n + case["block_items"] - 1) // case["block_items"]
        s["out"] = torch.empty((1 << case["bits"]) * m, dtype=torch.int64, device=DEVICE)
    else:
        s["out"] = torch.empty(n, dtype=binding.out_dtype(x, case["op"]), device=DEVICE)
    if kind == "batched":
        off = extra.tolist()
        ib, ob = x.element_size(), s["out"].element_size()
        s["table"] = binding.array_table([(x.data_ptr() + a * ib, s["out"].data_ptr() + a * ob, b - a)
                                          for a, b in zip(off[:-1], off[1:])])
        s["flags"] = ((binding.F_COMPENSATED if case["compensated"] else 0) |
                      (binding.F_EXCLUSIVE if case["exclusive"] else 0))
    return s


def run(s):
    case, kind = s["case"], s["kind"]
    if kind == "scan":
        call = binding.exclusive if case["exclusive"] else binding.inclusive
        return call(s["x"], case["op"], compensated=case["compensated"], out=s["out"])
    if kind == "segmented":
        return binding.segmented(s["x"], s["extra"], case["op"], exclusive=case["exclusive"],
                                 compensated=case["compensated"], out=s["out"])
    if kind == "batched":
        binding.lscan_batched(s["table"], binding.dtype_code(s["x"]), binding.OPS[case["op"]], s["flags"],
                              torch.cuda.current_stream().cuda_stream)
        return s["out"]
    if kind == "compact":
        return binding.compact(s["x"], s["extra"], out=s["out"], count=s["count"])
    if kind == "radix":
        return binding.radix_offsets(s["x"], case["shift"], case["bits"], case["block_items"], out=s["out"])
    # which parent a vertex gets is not fixed, so the searches ask for levels and totals
    levels, _, stats = binding.bfs(s["row"], s["col"], s["source"], levels=s["levels"], parents=False, stats=s["stats"])
    return levels, stats


def work(case):
    kind = case["kind"]
    if kind == "bfs":
        # rows read, levels written, every column entry read once (the largest component holds nearly all)
        nv = 1 << case["scale"]
        return {"bytes": 8 * (nv + 1) + 4 * nv + 4 * 2 * case["edge_factor"] * nv + 32, "flops": 0}
    n, ib = case["n"], IN_BYTES[case["dtype"]]
    if kind == "compact":
        kept = int(n * case["density"])
        return {"bytes": n * ib + (n if case["flags"] else 0) + kept * ib + 8, "flops": 0}
    if kind == "radix":
        m = (n + case["block_items"] - 1) // case["block_items"]
        return {"bytes": n * ib + 8 * (m << case["bits"]), "flops": n}
    extra = 8 * (case["segments"] + 1) if kind == "segmented" else 0
    return {"bytes": n * (ib + _out_bytes(case["dtype"], case["op"])) + extra, "flops": n}


def exact(case, seed):
    """Float results in float64 (whole-number results are the same in any order of combination)."""
    if case["kind"] not in ("scan", "segmented", "batched") or case["dtype"] not in ("float32", "bfloat16") or \
            case["op"] in ("argmax", "argmin"):
        return None
    x, off = _inputs(case, seed)
    x = x.double()
    if case["op"] == "add":
        y = torch.cumsum(x, 0)
        if off is not None:  # what lies before each element's segment
            lens = off[1:] - off[:-1]
            starts = torch.cat([torch.zeros(1, dtype=y.dtype, device=DEVICE), y])[off[:-1]]
            y -= torch.repeat_interleave(starts, lens)
        return y - x if case["exclusive"] else y
    if off is not None:
        return None
    empty = -math.inf if case["op"] == "max" else math.inf
    y = (torch.cummax(x, 0) if case["op"] == "max" else torch.cummin(x, 0)).values
    if case["exclusive"]:
        y = torch.cat([torch.full((1,), empty, dtype=y.dtype, device=DEVICE), y[:-1]])
    return y
