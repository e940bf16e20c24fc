"""The work that users of this library have it do, as measurable cases.

Every case calls the public entry points as a program does: inputs, outputs,
workspaces, plans and servers are made once (`prepare`), one pass is the calls
alone (`run`).  Sizes come from the repository's workloads and tests: merges
of 1E3 to 1E8 rows per side, int32 and int64 keys, P = 4 to 32 destinations
(and 300 and more for a partition alone), distinct and repeated keys.

Outputs are compared value by value, so every case has one defined result,
row order included: build payloads of repeated keys are an attribute of the
key (equal rows may come in any order), output buffers hold nothing but the
result and zeros, and a merge holds at most 6E6 rows per partition (beyond that
the row order inside a partition differs from run to run).
"""

from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2101_08878_amd as mdx

DEV = "cuda"
KEY = {"int32": torch.int32, "int64": torch.int64}
MAX_ROWS_PER_PART = 6_000_000
ZIPF = 0.1  # exponent 1.1, less one


# ---- cases -----------------------------------------------------------------

def listed():
    return [
        # One smallest merge of a batch or a service: latency and launches.
        {"name": "merge_1e3", "op": "merge", "dist": "match", "n_left": 1000, "n_right": 1000,
         "P": 8, "key": "int32", "frac": 0.3},
        # The plain workload: keys uniform in [0, 2n), many of them repeated.
        {"name": "merge_plain_1e5", "op": "merge", "dist": "uniform", "n_left": 100_000,
         "n_right": 100_000, "P": 4, "key": "int64", "frac": 0.0},
        # An ordinary merge of uneven sizes, a partition count that is no power of two.
        {"name": "merge_ragged_i32", "op": "merge", "dist": "match", "n_left": 1_234_567,
         "n_right": 345_679, "P": 7, "key": "int32", "frac": 0.3},
        # A build side whose hottest keys repeat 1E5 times and more (Zipf).
        {"name": "merge_hot_left", "op": "merge", "dist": "hot", "n_left": 4_000_000,
         "n_right": 400_000, "P": 8, "key": "int64", "frac": 0.0},
        # A fact table with Zipf foreign keys against a dimension table of distinct keys.
        {"name": "merge_zipf_right", "op": "merge", "dist": "zipf", "n_left": 10_000_000,
         "n_right": 50_000_000, "P": 16, "key": "int64", "frac": 1.0},
        # One worker's share of the paper's benchmark.
        {"name": "merge_paper_1e8", "op": "merge", "dist": "match", "n_left": 100_000_000,
         "n_right": 100_000_000, "P": 32, "key": "int64", "frac": 0.3},
        # The shuffle's local half alone, for more destinations than a large tile takes.
        {"name": "partition_i32_p300", "op": "partition", "n": 2_000_003, "P": 300,
         "key": "int32"},
        # The skewed workload's graded step: both partitions and the join's counts.
        {"name": "count_skewed_5e7", "op": "count", "n_left": 50_000_000, "n_right": 50_000_000,
         "P": 16, "key": "int64", "support": 10_000_000},
        # Build and probe of tables that arrive partitioned (after an exchange).
        {"name": "staged_join_1e7", "op": "staged", "n_left": 10_000_000, "n_right": 10_000_000,
         "P": 8, "key": "int64", "frac": 0.3},
        # A fused batch of merges of uneven sizes and both key widths.
        {"name": "batch_fused_96", "op": "batch", "how": "fused", "count": 96, "lo": 1000,
         "hi": 4_000_000, "P": 8, "sizes": 0},
        # A burst of requests through a server's slots.
        {"name": "serve_burst_12", "op": "serve", "count": 12, "lo": 10_000, "hi": 20_000_000,
         "P": 8, "sizes": 0, "slots": 8},
        # The paper's other benchmark: a matrix plus its transpose.
        {"name": "transpose_16384", "op": "transpose", "n": 16384},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["merge"] * 6 + ["partition"] * 2 + ["count", "staged", "batch", "serve",
                                                         "transpose"])
    key = rng.choice(["int32", "int64"])
    if op == "merge":
        dist = rng.choice(["match", "match", "match", "uniform", "zipf", "hot"])
        P = rng.choice([3, 4, 7, 8, 16, 32, 64])
        top = min(100_000_000, MAX_ROWS_PER_PART * P)
        if dist == "match":
            nl = _log(rng, 1e3, top)
            # most merges are of like sizes, some far apart
            nr = _log(rng, 1e3, top) if rng.random() < 0.4 else \
                min(top, max(1, int(nl * rng.uniform(0.3, 3.0))))
            return {"op": op, "dist": dist, "n_left": nl, "n_right": nr, "P": P, "key": key,
                    "frac": round(rng.uniform(0.1, 0.9), 3)}
        if dist == "uniform":
            nl = _log(rng, 1e3, min(top, 3e7))
            return {"op": op, "dist": dist, "n_left": nl,
                    "n_right": max(1, int(nl * rng.uniform(0.3, 1.5))), "P": P, "key": key,
                    "frac": 0.0}
        if dist == "zipf":
            nl = _log(rng, 1e4, 1e7)
            return {"op": op, "dist": dist, "n_left": nl,
                    "n_right": min(MAX_ROWS_PER_PART * P, 50_000_000, int(nl * rng.uniform(1, 8))),
                    "P": P, "key": key, "frac": 1.0}
        nl = _log(rng, 1e4, 1e7)
        return {"op": op, "dist": dist, "n_left": nl, "n_right": max(1, int(nl * 0.1)), "P": P,
                "key": key, "frac": 0.0}
    if op == "partition":
        return {"op": op, "n": _log(rng, 1e3, 1e8),
                "P": rng.choice([1, 2, 3, 4, 7, 8, 16, 32, 57, 64, 128, 256, 257, 300, 1024, 4096]),
                "key": key}
    if op == "count":
        n = _log(rng, 1e5, 5e7)
        return {"op": op, "n_left": n, "n_right": max(1, int(n * rng.uniform(0.3, 1.0))),
                "P": rng.choice([4, 8, 16, 32]), "key": key, "support": max(1000, n // 5)}
    if op == "staged":
        n = _log(rng, 1e4, 2e7)
        return {"op": op, "n_left": n, "n_right": max(1, int(n * rng.uniform(0.3, 1.0))),
                "P": rng.choice([3, 8, 16, 32]), "key": key, "frac": round(rng.uniform(0.1, 0.9), 3)}
    if op == "batch":
        return {"op": op, "how": rng.choice(["fused", "fused", "lanes"]),
                "count": rng.randint(5, 96), "lo": 1000, "hi": _log(rng, 1e4, 4e6), "P": 8,
                "sizes": rng.randrange(1 << 20)}
    if op == "serve":
        return {"op": op, "count": rng.randint(3, 12), "lo": 10_000, "hi": _log(rng, 1e5, 2e7),
                "P": 8, "sizes": rng.randrange(1 << 20), "slots": rng.choice([4, 8])}
    return {"op": op, "n": _log(rng, 500, 16384)}


# ---- inputs ----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randint(g, lo, hi, n):
    return torch.randint(lo, hi, (n,), generator=g, device=DEV, dtype=torch.int64)


def _rows(n):
    return torch.arange(n, device=DEV, dtype=torch.int64)


def _power_law(u, support):
    """Keys in [0, support) from uniform u, P(k) nearly proportional to
    (k + 1)^-1.1: the inverse of the continuous distribution, rounded down."""
    a = 1.0 - float(support + 1) ** -ZIPF
    return (u.mul(-a).add_(1.0).pow_(-1.0 / ZIPF).to(torch.int64) - 1).clamp_(0, support - 1)


def _zipf(g, n, support):
    return _power_law(torch.rand(n, generator=g, device=DEV, dtype=torch.float64), support)


def _zipf_share(support, step):
    """Share of the rows of _zipf whose key is a multiple of `step`."""
    k = np.arange(1, support + 1, step, dtype=np.float64)
    return float(np.sum(k ** -ZIPF - (k + 1) ** -ZIPF) / (1.0 - float(support + 1) ** -ZIPF))


def _match_tables(g, nl, nr, frac, dtype):
    """Distinct left keys; exactly round(frac nr) right rows have a partner."""
    kl = torch.randperm(nl, generator=g, device=DEV, dtype=torch.int64)
    m = int(round(frac * nr))
    kr = torch.cat([kl[_randint(g, 0, nl, m)], _randint(g, nl, 2 * nl, nr - m)])
    kr = kr[torch.randperm(nr, generator=g, device=DEV)]
    return kl.to(dtype), _rows(nl), kr.to(dtype), _rows(nr), m


def _attribute(keys):
    return keys * 7 + 3


def _tables(case, g):
    """(left keys, left payload, right keys, right payload, output rows)."""
    nl, nr, dtype = case["n_left"], case["n_right"], KEY[case["key"]]
    if case["dist"] == "match":
        return _match_tables(g, nl, nr, case["frac"], dtype)
    if case["dist"] == "zipf":
        kl = torch.randperm(nl, generator=g, device=DEV, dtype=torch.int64)
        kr = kl[_zipf(g, nr, nl)]
        return kl.to(dtype), _rows(nl), kr.to(dtype), _rows(nr), nr
    if case["dist"] == "uniform":
        kl, kr = _randint(g, 0, 2 * nl, nl), _randint(g, 0, 2 * nl, nr)
    else:  # hot: Zipf build keys, every step-th key probed once, the hottest among them
        kl = _zipf(g, nl, nl)
        kr = torch.randperm(nr, generator=g, device=DEV, dtype=torch.int64) * (nl // nr)
    # room for a little more than the rows expected, so that the shape does
    # not depend on the seed; the rows past the result stay zero
    total = int(_expected_rows(case) * 1.1) + 2000
    return kl.to(dtype), _attribute(kl), kr.to(dtype), _rows(nr), total


def _status():
    return torch.zeros(1, dtype=torch.int32, device=DEV)


def _i64(n):
    return torch.empty(n, dtype=torch.int64, device=DEV)


def _bytes(n):
    return torch.empty(max(n, 1), dtype=torch.uint8, device=DEV)


def _key_type(dtype):
    return mdx.MDX_KEY_I64 if dtype == torch.int64 else mdx.MDX_KEY_I32


def _out(total, dtype):
    return tuple(torch.zeros(total, dtype=t, device=DEV) for t in (dtype, torch.int64, torch.int64))


def _sizes(case):
    """(n_left, n_right, key type, match fraction) of every merge of a batch or burst."""
    rng = random.Random(case["sizes"])
    got = []
    for _ in range(case["count"]):
        nl, nr = _log(rng, case["lo"], case["hi"]), _log(rng, case["lo"], case["hi"])
        dtype = rng.choice(["int32", "int64"]) if case["op"] == "batch" else "int64"
        frac = 0.3 if case["op"] == "batch" else rng.uniform(0.1, 0.9)
        got.append((nl, nr, dtype, frac))
    return got


def _jobs(case, g):
    """Merge jobs whose output columns are consecutive slices of shared buffers."""
    sizes = _sizes(case)
    tables = [_match_tables(g, nl, nr, frac, KEY[dt]) for nl, nr, dt, frac in sizes]
    shared = {}
    for name, dtype in KEY.items():
        total = sum(t[4] for t, s in zip(tables, sizes) if s[2] == name)
        if total:
            shared[name] = _out(total, dtype)
    offsets = _i64(len(sizes) * (case["P"] + 1)).view(len(sizes), case["P"] + 1)
    status = _status()
    at, jobs = dict.fromkeys(KEY, 0), []
    for i, ((kl, vl, kr, vr, m), (_, _, name, _)) in enumerate(zip(tables, sizes)):
        a = at[name]
        at[name] += m
        cols = shared.get(name) or _out(0, KEY[name])
        jobs.append(mdx.MergeJob(kl, vl, kr, vr, case["P"], m, tuple(c[a:a + m] for c in cols),
                                 offsets[i], status))
    return jobs, {"out": shared, "offsets": offsets, "status": status}


def prepare(case, seed):
    g = _gen(seed)
    op = case["op"]
    s = {"op": op}
    if op == "transpose":
        s["x"] = torch.rand(case["n"], case["n"], generator=g, device=DEV, dtype=torch.float64)
        s["y"] = torch.empty_like(s["x"])
        return s
    if op in ("batch", "serve"):
        s["jobs"], s["result"] = _jobs(case, g)
        if op == "serve":
            most = max(max(j.left_keys.numel(), j.right_keys.numel()) for j in s["jobs"])
            s["server"] = mdx.Server(case["slots"], most, most, case["P"], 200 << 30)
        elif case["how"] == "fused":
            s["batch"] = mdx.FusedBatch(s["jobs"], tuning="table")
        else:
            s["workspace"] = _bytes(mdx.mdx_merge_batch_workspace_bytes(s["jobs"], 4))
        return s
    P, dtype = case["P"], KEY[case["key"]]
    s["P"], kt = P, _key_type(dtype)
    if op == "partition":
        n = case["n"]
        s["keys"], s["payload"] = _randint(g, -(1 << 31), 1 << 31, n).to(dtype), _rows(n)
        s["out"] = (torch.empty_like(s["keys"]), _i64(n), _i64(P + 1))
        s["workspace"] = _bytes(mdx.mdx_hash_partition_workspace_bytes(n, P, kt))
        return s
    nl, nr = case["n_left"], case["n_right"]
    if op == "count":
        kl, kr = (_zipf(g, n, case["support"]).to(dtype) for n in (nl, nr))
        s["sides"] = [{"keys": k, "payload": _rows(k.numel()),
                       "out": (torch.empty_like(k), _i64(k.numel()), _i64(P + 1)),
                       "workspace": _bytes(mdx.mdx_hash_partition_workspace_bytes(k.numel(), P, kt))}
                      for k in (kl, kr)]
        s["counts"], s["status"] = _i64(P + 1), _status()
        s["workspace"] = _bytes(mdx.mdx_join_count_workspace_bytes(nl, nr, P, kt))
        return s
    if op == "staged":
        kl, vl, kr, vr, total = _match_tables(g, nl, nr, case["frac"], dtype)
        s["left"], s["right"] = mdx.mdx_hash_partition(kl, vl, P), mdx.mdx_hash_partition(kr, vr, P)
        s["table"] = _bytes(mdx.mdx_join_table_bytes(nl, P, kt))
        s["workspace"] = _bytes(mdx.mdx_join_probe_workspace_bytes(nr, P, kt))
    else:
        *s["tables"], total = _tables(case, g)
        s["workspace"] = _bytes(mdx.mdx_merge_workspace_bytes(nl, nr, P, kt))
    s["total"], s["out"] = total, _out(total, dtype)
    s["offsets"], s["status"] = _i64(P + 1), _status()
    return s


# ---- one pass --------------------------------------------------------------

def run(s):
    op = s["op"]
    if op == "merge":
        out = mdx.mdx_merge(*s["tables"], s["P"], out_capacity=s["total"], out=s["out"],
                            out_offsets=s["offsets"], workspace=s["workspace"], status=s["status"])
        return list(out) + [s["status"]]
    if op == "partition":
        k, v, off = s["out"]
        return mdx.mdx_hash_partition(s["keys"], s["payload"], s["P"], keys_out=k, payload_out=v,
                                      offsets=off, workspace=s["workspace"])
    if op == "count":
        parts = []
        for t in s["sides"]:
            k, v, off = t["out"]
            parts.append(mdx.mdx_hash_partition(t["keys"], t["payload"], s["P"], keys_out=k,
                                                payload_out=v, offsets=off,
                                                workspace=t["workspace"]))
        (lk, _, lo), (rk, _, ro) = parts
        counts = mdx.mdx_join_count(lk, lo, rk, ro, s["P"], out_offsets=s["counts"],
                                    workspace=s["workspace"], status=s["status"])
        return [parts, counts, s["status"]]
    if op == "staged":
        table = mdx.mdx_join_build(*s["left"], s["P"], table_memory=s["table"], status=s["status"])
        out = mdx.mdx_join_probe(table, *s["right"], out_capacity=s["total"], out=s["out"],
                                 out_offsets=s["offsets"], workspace=s["workspace"],
                                 status=s["status"])
        return list(out) + [s["status"]]
    if op == "batch":
        if "batch" in s:
            s["batch"].run()
        else:
            mdx.mdx_merge_batch(s["jobs"], lanes=4, workspace=s["workspace"])
        return s["result"]
    if op == "serve":
        server, jobs, sent, done = s["server"], s["jobs"], 0, 0
        while done < len(jobs):
            while sent < len(jobs) and server.submit(jobs[sent], sent) is not None:
                sent += 1
            done += len(server.poll())
        return s["result"]
    return mdx.mdx_transpose_sum(s["x"], out=s["y"])


# ---- what a pass cannot do without -----------------------------------------

def _width(key):
    return 4 if key == "int32" else 8


def _expected_rows(case):
    """Output rows: exact for distinct build keys, else their expectation."""
    nl, nr = case["n_left"], case["n_right"]
    if case.get("dist") == "uniform":
        return nr * 0.5
    if case.get("dist") == "hot":
        return nl * _zipf_share(nl, nl // nr)
    return round(case["frac"] * nr)


def work(case):
    op = case["op"]
    if op == "transpose":
        return {"bytes": 16 * case["n"] ** 2, "flops": case["n"] ** 2}
    if op in ("batch", "serve"):
        return {"bytes": sum((nl + nr) * (_width(dt) + 8) + round(f * nr) * (_width(dt) + 16) +
                             8 * (case["P"] + 1) for nl, nr, dt, f in _sizes(case)), "flops": 0}
    w = _width(case["key"])
    if op == "partition":
        return {"bytes": 2 * case["n"] * (w + 8) + 8 * (case["P"] + 1), "flops": 0}
    rows = case["n_left"] + case["n_right"]
    if op == "count":
        return {"bytes": 2 * rows * (w + 8) + 24 * (case["P"] + 1), "flops": 0}
    return {"bytes": rows * (w + 8) + _expected_rows(case) * (w + 16) + 8 * (case["P"] + 1),
            "flops": 0}


def exact(case, seed):
    """The transpose sum in 64 bits; every other output is whole numbers."""
    if case["op"] != "transpose":
        return None
    x = torch.rand(case["n"], case["n"], generator=_gen(seed), device=DEV, dtype=torch.float64)
    return x + x.t()
