"""The calls that are timed: flat and v-way partition, filter, segmented
partition, the segment helpers, the differentiable partition, the property
checks and get_smallest_pairs, each through the package's public functions.

Sizes are those of bench.py, the tests and the paper's evaluation (50M-200M
random floats; 10^4 log-normal rows; 2^26 graph entries), rounded to odd
numbers where a program would have no reason to hold a round one.  All inputs
are drawn on the GPU from the seed alone.
"""
import math

import torch

import paper_2506_23058_amd as P

DEV = "cuda"
IDX = {"int32": torch.int32, "int64": torch.int64}
MODE = {"partition": P.MODE_PARTITION, "filter": P.MODE_FILTER}


def listed():
    return [
        # the smallest call: one partition step inside a larger program, where
        # launches and the host path are all there is
        {"name": "partition_tiny", "op": "flat", "mode": "partition", "n": 4099, "pred": "mod", "p": 2,
         "idx": "int64"},
        # an ordinary array of integers, parity split, default 64-bit indices
        {"name": "partition_1m", "op": "flat", "mode": "partition", "n": 1 << 20, "pred": "mod", "p": 2,
         "idx": "int64"},
        # the headline workload of bench.py
        {"name": "partition_256m", "op": "flat", "mode": "partition", "n": 1 << 28, "pred": "lt", "p": 0.5,
         "idx": "int32"},
        # filter of the paper's 100M floats
        {"name": "filter_100m", "op": "flat", "mode": "filter", "n": 100_000_003, "pred": "lt", "p": 0.5,
         "idx": "int32"},
        # partition3 of the paper's 50M floats
        {"name": "partition3_50m", "op": "vway", "n": 50_000_017, "cls": "thresh", "v": 3, "idx": "int32"},
        # partition2L of thousands of uneven rows (bench.py's jagged array)
        {"name": "segmented_10k_rows", "op": "seg", "mode": "partition", "n": 70_386_872, "m": 10_000,
         "pred": "mod", "p": 3, "empty": 0.0, "idx": "int32", "descr": True},
        # partition2L of many short rows, some of them empty, such as the
        # adjacency lists of a sparse graph, by a threshold of each row
        {"name": "segmented_short_rows", "op": "seg", "mode": "partition", "n": 8_000_011, "m": 250_007,
         "pred": "lt_rows", "p": 0, "empty": 0.1, "idx": "int32", "descr": False},
        # the flat-form helpers of a jagged array: row numbers, a descriptor
        # and a running sum that restarts at every row
        {"name": "segment_helpers", "op": "helpers", "n": 33_554_467, "m": 100_003, "empty": 0.1, "ii": "int32"},
        # forward and backward of a payload of 16 floats moved with its keys
        {"name": "differentiable_4m_rows", "op": "autograd", "mode": "partition", "n": (1 << 22) + 3, "width": 16},
        # a permutation checked before it is used as scatter indices
        {"name": "check_permutation_128m", "op": "perm", "n": 1 << 27, "x": "int64", "faults": 0},
        # a partition's outputs checked against their definition
        {"name": "check_filtpart_16m", "op": "filtpart", "mode": "partition", "n": (1 << 24) + 5, "pred": "mod",
         "p": 3, "idx": "int32", "faults": 0},
        # get_smallest_pairs of maximal matching, bench.py's size
        {"name": "smallest_pairs_64m", "op": "pairs", "n": 1 << 26, "verts": 1 << 24},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _flat_pred(rng):
    pred = rng.choice(["mod", "lt", "lt", "flags"])
    return {"pred": pred, "p": {"mod": rng.choice([2, 3, 7, 10]), "lt": rng.choice([0.01, 0.25, 0.5, 0.99]),
                                "flags": rng.choice([0.1, 0.5, 0.9])}[pred]}


def draw(rng):
    op = rng.choice(["flat", "flat", "flat", "vway", "seg", "seg", "seg", "helpers", "autograd", "perm", "filtpart",
                     "pairs"])
    if op == "flat":
        return {"op": op, "mode": rng.choice(["partition", "partition", "filter"]), "n": _log(rng, 1000, 1 << 28),
                "idx": rng.choice(["int32", "int64"]), **_flat_pred(rng)}
    if op == "vway":
        return {"op": op, "n": _log(rng, 1 << 14, 200_000_000), "cls": rng.choice(["thresh", "mod", "bytes"]),
                "v": rng.choice([2, 3, 3, 4]), "idx": rng.choice(["int32", "int64"])}
    if op == "seg":
        m = _log(rng, 30, 1_000_000)
        n = min(m * _log(rng, 6, 1 << 16), _log(rng, 1 << 22, 1 << 27))
        pred = rng.choice(["mod", "mod", "lt_rows", "flags"])
        return {"op": op, "mode": rng.choice(["partition", "partition", "filter"]), "n": n, "m": m, "pred": pred,
                "p": {"mod": rng.choice([2, 3, 10]), "lt_rows": 0, "flags": 0.5}[pred],
                "empty": rng.choice([0.0, 0.1, 0.5]), "idx": rng.choice(["int32", "int64"]),
                "descr": rng.choice([True, False])}
    if op == "helpers":
        m = _log(rng, 100, 1_000_000)
        return {"op": op, "n": min(m * _log(rng, 6, 1 << 14), _log(rng, 1 << 20, 1 << 26)), "m": m,
                "empty": rng.choice([0.0, 0.1]), "ii": rng.choice(["int32", "int64"])}
    if op == "autograd":
        width = rng.choice([1, 3, 4, 8, 16, 24, 32, 64])
        return {"op": op, "mode": rng.choice(["partition", "partition", "filter"]),
                "n": _log(rng, 1000, (1 << 26) // width), "width": width}
    if op == "perm":
        return {"op": op, "n": _log(rng, 1 << 12, 1 << 27), "x": rng.choice(["int64", "int64", "int32"]),
                "faults": rng.choice([0, 0, 0, 1, 100])}
    if op == "filtpart":
        return {"op": op, "mode": rng.choice(["partition", "partition", "filter"]), "n": _log(rng, 1 << 12, 1 << 25),
                "idx": rng.choice(["int32", "int64"]), "faults": rng.choice([0, 0, 0, 1]), **_flat_pred(rng)}
    n = _log(rng, 1 << 14, 1 << 26)
    return {"op": op, "n": n, "verts": max(1, int(n / rng.uniform(2, 16)))}


# ------------------------------------------------------------------- inputs --

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _int_keys(n, g):
    return torch.randint(0, (1 << 31) - 1, (n,), dtype=torch.int32, device=DEV, generator=g)


def _f32_keys(n, g):
    return torch.rand(n, dtype=torch.float32, device=DEV, generator=g)


def _keys_and_pred(case, n, g, m=0):
    """Keys and predicate, and what exact() needs of them."""
    kind = case["pred"]
    if kind == "mod":
        return _int_keys(n, g), P.Pred.mod_eq(case["p"], 0), None
    keys = _f32_keys(n, g)
    if kind == "lt":
        return keys, P.Pred.lt(case["p"]), None
    if kind == "flags":
        flags = (torch.rand(n, device=DEV, generator=g) < case["p"]).to(torch.uint8)
        return keys, P.Pred.from_flags(flags), flags
    row_s = torch.rand(m, dtype=torch.float32, device=DEV, generator=g)
    return keys, P.Pred.lt_rows(row_s), row_s


def _shape(n, m, empty, g):
    """m row sizes that sum to n: log-normal (sigma 1.5 in log2), a share of them empty."""
    w = torch.exp2(1.5 * torch.randn(m, dtype=torch.float64, device=DEV, generator=g))
    if empty:
        gone = torch.rand(m, device=DEV, generator=g) < empty
        gone[0] = False
        w[gone] = 0.0
    end = torch.round(torch.cumsum(w, 0) / w.sum() * n).to(torch.int64)
    end[-1] = n
    return torch.diff(end, prepend=torch.zeros(1, dtype=torch.int64, device=DEV))


def _faulty(x, k, g):
    """k entries of x overwritten with copies of other entries."""
    n = x.numel()
    if k:
        at = torch.randint(0, n, (2 * k,), device=DEV, generator=g)
        x[at[:k]] = x[at[k:]]
    return x


def _classes(case, n, g):
    v = case["v"]
    if case["cls"] == "mod":
        return _int_keys(n, g), P.Classes.mod(v), None
    keys = _f32_keys(n, g)
    if case["cls"] == "thresh":
        return keys, P.Classes.thresholds(*[k / v for k in range(1, v)]), None
    cls = torch.randint(0, v, (n,), dtype=torch.uint8, device=DEV, generator=g)
    return keys, P.Classes.from_bytes(cls, v), cls


def prepare(case, seed):
    g, op, n = _gen(seed), case["op"], case["n"]
    s = {"case": case}
    if op == "flat":
        s["keys"], s["pred"], s["extra"] = _keys_and_pred(case, n, g)
        # a filter writes only the kept part of its output: the program's own, cleared buffer
        s["out"] = torch.zeros_like(s["keys"]) if case["mode"] == "filter" else None
    elif op == "vway":
        s["keys"], s["classes"], s["extra"] = _classes(case, n, g)
    elif op == "seg":
        s["shape"] = _shape(n, case["m"], case["empty"], g)
        s["keys"], s["pred"], s["extra"] = _keys_and_pred(case, n, g, case["m"])
        s["out"] = torch.zeros_like(s["keys"]) if case["mode"] == "filter" else None
    elif op == "helpers":
        s["shape"] = _shape(n, case["m"], case["empty"], g)
        s["xs"] = torch.randint(1, 1 << 40, (case["m"],), device=DEV, generator=g)
        s["vals"] = torch.randint(0, 1 << 31, (n,), dtype=torch.int64, device=DEV, generator=g)
        ends = torch.cumsum(s["shape"], 0)
        starts = (ends - s["shape"])[s["shape"] > 0]
        s["flags"] = torch.zeros(n, dtype=torch.uint8, device=DEV)
        s["flags"][starts] = 1
    elif op == "autograd":
        s["keys"], s["pred"] = _int_keys(n, g), P.Pred.mod_eq(2, 0)
        s["payload"] = torch.randn((n, case["width"]), device=DEV, generator=g).requires_grad_(True)
        s["gy"] = torch.randn((n, case["width"]), device=DEV, generator=g)
    elif op == "perm":
        s["x"] = _faulty(torch.randperm(n, device=DEV, generator=g).to(IDX[case["x"]]), case["faults"], g)
    elif op == "filtpart":
        s["keys"], s["pred"], s["extra"] = _keys_and_pred(case, n, g)
        out, idx, split = P.partition(s["keys"], s["pred"], MODE[case["mode"]], IDX[case["idx"]])
        s["x"] = _faulty(idx, case["faults"], g)
        s["fp"] = P.FiltPartArgs(s["keys"], out, s["pred"], split, MODE[case["mode"]])
    else:
        es = torch.randint(0, case["verts"], (n,), device=DEV, generator=g)
        s["pairs"] = P.SmallestPairs(case["verts"], n, es, torch.randperm(n, device=DEV, generator=g))
        s["pairs"].es_out.zero_()   # past the kept pairs nothing is written
        s["pairs"].is_out.zero_()
    return s


# --------------------------------------------------------------------- calls --

def run(s):
    case, op = s["case"], s["case"]["op"]
    if op == "flat":
        return P.partition(s["keys"], s["pred"], MODE[case["mode"]], IDX[case["idx"]], out_keys=s["out"])
    if op == "vway":
        return P.partition_v(s["keys"], s["classes"], IDX[case["idx"]])
    if op == "seg":
        return P.segmented_partition(s["keys"], s["shape"], s["pred"], MODE[case["mode"]], IDX[case["idx"]],
                                     want_flags=case["descr"], out_keys=s["out"])
    if op == "helpers":
        return (P.mk_ii(s["shape"], case["n"], IDX[case["ii"]]), P.mk_sgm_descr(s["shape"], s["xs"], case["n"]),
                P.sgm_sum(s["flags"], s["vals"]))
    if op == "autograd":
        y, keys, idx, split = P.partition_scatter(s["keys"], s["payload"], s["pred"], MODE[case["mode"]])
        grad, = torch.autograd.grad(y, s["payload"], s["gy"])
        if case["mode"] == "filter":
            return y.detach(), idx, split, grad   # the keys past the kept ones are not written
        return y.detach(), keys, idx, split, grad
    if op == "perm":
        n = case["n"]   # the checked array goes on with its verdicts
        return s["x"], P.check_props(s["x"], P.RANGE | P.INJ | P.BIJ, lo=0, hi=n, img_lo=0, img_hi=n)
    if op == "filtpart":
        return s["x"], P.check_props(s["x"], P.FILTPART, fp=s["fp"])
    return s["pairs"].run()


def work(case):
    """Bytes each input and output needs once; there is no arithmetic to speak of."""
    op, n = case["op"], case["n"]
    isz = {"int32": 4, "int64": 8}.get(case.get("idx"), 4)
    if op in ("flat", "seg"):
        if case["pred"] == "mod":
            kept = 1.0 / case["p"]
        else:
            kept = 0.5 if case["pred"] == "lt_rows" else case["p"]
        out = 4 * kept if case["mode"] == "filter" else 4
        b = n * (4 + isz + out + (1 if case["pred"] == "flags" else 0))
        if op == "seg":
            b += case["m"] * (16 + (4 if case["pred"] == "lt_rows" else 0)) + (n if case["descr"] else 0)
        return {"bytes": b, "flops": 0}
    if op == "vway":
        return {"bytes": n * (8 + isz + (1 if case["cls"] == "bytes" else 0)), "flops": 0}
    if op == "helpers":
        return {"bytes": n * ((4 if case["ii"] == "int32" else 8) + 8 + 17) + case["m"] * 24, "flops": 0}
    if op == "autograd":
        row = 4 * case["width"]
        return {"bytes": n * (12 + 2 * (4 + 2 * row)), "flops": 0}
    if op == "perm":
        return {"bytes": n * (8 if case["x"] == "int64" else 4), "flops": 0}
    if op == "filtpart":
        kept = 1.0
        if case["mode"] == "filter":
            kept = 1.0 / case["p"] if case["pred"] == "mod" else case["p"]
        return {"bytes": n * (isz + 4 + 4 * kept + (1 if case["pred"] == "flags" else 0)), "flops": 0}
    kept = case["verts"] * (1 - math.exp(-n / case["verts"]))
    return {"bytes": 16 * n + 16 * kept, "flops": 0}


# --------------------------------------------------------------------- exact --

def _flags_of(s, row=None):
    case, keys = s["case"], s["keys"]
    if case["pred"] == "mod":
        return torch.remainder(keys, case["p"]) == 0
    if case["pred"] == "lt":
        return keys < torch.tensor(case["p"], dtype=torch.float32, device=DEV)
    if case["pred"] == "flags":
        return s["extra"] != 0
    return keys < s["extra"][row]


def _rows(shape):
    return torch.repeat_interleave(torch.arange(shape.numel(), device=DEV), shape)


def _filtered(keys, c):
    out = torch.zeros_like(keys)
    kept = keys[c]
    out[:kept.shape[0]] = kept
    return out


def _verdicts(properties):
    return torch.tensor([[1, -1, 0]] * properties, device=DEV)   # every one holds


def exact(case, seed):
    s, op, n = prepare(case, seed), case["op"], case["n"]
    if op in ("flat", "autograd"):
        c = torch.remainder(s["keys"], 2) == 0 if op == "autograd" else _flags_of(s)
        before = torch.cumsum(c, 0) - c.to(torch.int64)
        t = c.sum().reshape(1)
        if case["mode"] == "filter":
            idx = torch.where(c, before, -1)
            keys = _filtered(s["keys"], c)
        else:
            idx = torch.where(c, before, t + torch.arange(n, device=DEV) - before)
            keys = torch.cat([s["keys"][c], s["keys"][~c]])
        if op == "flat":
            return keys, idx, t
        x, gy = s["payload"].detach(), s["gy"]
        if case["mode"] == "filter":
            return _filtered(x, c), idx, t, torch.where(c[:, None], gy[idx.clamp(min=0)], 0.0)
        return torch.cat([x[c], x[~c]]), keys, idx, t, gy[idx]
    if op == "vway":
        v, k = case["v"], s["keys"]
        if case["cls"] == "mod":
            cls = torch.remainder(k, v).to(torch.int64)
        elif case["cls"] == "bytes":
            cls = s["extra"].to(torch.int64)
        else:
            cls = torch.zeros(n, dtype=torch.int64, device=DEV)
            for j in range(1, v):
                cls += k >= torch.tensor(j / v, dtype=torch.float32, device=DEV)
        idx, base, counts, parts = torch.empty(n, dtype=torch.int64, device=DEV), 0, [], []
        for j in range(v):
            c = cls == j
            idx[c] = base + torch.arange(int(c.sum()), device=DEV)
            counts.append(int(c.sum()))
            parts.append(k[c])
            base += counts[-1]
        return torch.cat(parts), idx, torch.tensor(counts, device=DEV)
    if op == "seg":
        shape, m = s["shape"], case["m"]
        row = _rows(shape)
        c = _flags_of(s, row)
        t = torch.zeros(m, dtype=torch.int64, device=DEV).index_add_(0, row, c.to(torch.int64))
        before = torch.cumsum(c, 0) - c.to(torch.int64)
        off = torch.cumsum(shape, 0) - shape
        descr = None
        if case["descr"]:
            descr = torch.zeros(n, dtype=torch.uint8, device=DEV)
            descr[off[shape > 0]] = 1
        if case["mode"] == "filter":
            return _filtered(s["keys"], c), torch.where(c, before, -1), t, descr
        in_row = before - (torch.cumsum(t, 0) - t)[row]
        o = off[row]
        idx = torch.where(c, o + in_row, t[row] + torch.arange(n, device=DEV) - in_row)
        return torch.empty_like(s["keys"]).index_copy_(0, idx, s["keys"]), idx, t, descr
    if op == "helpers":
        shape, vals = s["shape"], s["vals"]
        row = _rows(shape)
        off = torch.cumsum(shape, 0) - shape
        descr = torch.zeros(n, dtype=torch.int64, device=DEV)
        descr[off[shape > 0]] = s["xs"][shape > 0]
        run_sum = torch.cumsum(vals, 0)
        before = run_sum - vals
        return row, descr, run_sum - before[off[row]]
    if op in ("perm", "filtpart"):
        return s["x"], None if case["faults"] else _verdicts(5)
    es, ids = s["pairs"].es, s["pairs"].is_
    least = torch.full((case["verts"],), n, dtype=torch.int64, device=DEV)
    least.scatter_reduce_(0, es, ids, "amin")
    c = least[es] == ids
    return _filtered(es, c), _filtered(ids, c), c.sum().reshape(1)
