"""Workloads of the library, as its users run them, for timing.

Every case is one pass through the public entry points on inputs that are already on the device: bulk
and single-batch lookups, multi-request lookups, builds from a thousand to 100 million keys over the
bucket sizes, codings, load factors and partition sizes in use, string keys, batched builds, loading a
saved image, and the serving loop. A build's result is the table it makes, so build cases return the
positions of all their keys (and the size of the structure); all outputs are whole numbers.

``work`` counts each input byte read once and each output byte written once. The pilot search has no
closed operation count and is integer work, so no floating-point operations are stated.
"""

import math

import numpy as np
import torch

import paper_2404_18497_amd as phobic

LOOKUPS = 1_000_000


def listed():
    return [
        # a service looks up a handful of keys at a time: the launch itself counts
        dict(name="query_small", kind="query", n=1_000_000, q=1_000, lam=7.0, coding="rice", n_compact=0),
        # one batch of a bulk lookup stream against the full-size table
        dict(name="query_batch", kind="query", n=100_000_000, q=LOOKUPS, lam=7.0, coding="rice", n_compact=0),
        # a front end collects the requests of many clients against several resident tables
        dict(name="query_multi", kind="multi", tables=16, n=500_000, requests=64, q_lo=1_000, q_hi=300_000, lam=7.0,
             mix=1),
        # the smallest table of the batched workload, built alone
        dict(name="build_tiny", kind="build", n=1_000, lam=7.0, P=2500, coding="rice", bucket_fn="optimized",
             order="random"),
        # an ordinary index, with the larger buckets and the faster coding
        dict(name="build_medium", kind="build", n=1_300_021, lam=9.0, P=2500, coding="compact",
             bucket_fn="optimized", order="random"),
        # the headline size
        dict(name="build_large", kind="build", n=100_000_000, lam=7.0, P=2500, coding="rice",
             bucket_fn="optimized", order="random"),
        # the space-optimised setting: large buckets, nearly all time in the pilot search
        dict(name="build_dense", kind="build", n=400_009, lam=12.0, P=2500, coding="rice", bucket_fn="optimized",
             order="random"),
        # large partitions, for fewer offsets and better coding
        dict(name="build_wide", kind="build", n=10_000_000, lam=7.0, P=50_000, coding="rice",
             bucket_fn="optimized", order="random"),
        # string keys with a load factor below one and the remap table
        dict(name="build_strings", kind="strings", n=10_000_000, lam=7.0, coding="rice", alpha_num=99, alpha_den=100,
             lo=10, hi=50),
        # many independent tables of uneven sizes in one call (one per shard or column)
        dict(name="build_batch", kind="batch", count=512, median=50_000, lam=7.0, mix=5),
        # a program starts: reads a saved table and answers its first batch
        dict(name="load", kind="load", n=10_000_000, q=LOOKUPS, lam=7.0, coding="rice"),
        # the serving loop: queries against resident tables with builds among them
        dict(name="serve", kind="serve", tables=8, n=500_000, queries=60, q_lo=1_000, q_hi=1_000_000, builds=6,
             median=500_000, lam=7.0, mix=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query", "query", "multi", "build", "build", "build", "build", "wide", "dense", "strings",
                       "batch", "load", "serve"])
    coding = rng.choice(["rice", "rice", "compact"])
    if kind == "query":
        c = rng.choice([0, 0, 16, 64]) if coding == "rice" else 0
        return dict(kind=kind, n=_log_int(rng, 10_000, 100_000_000), q=_log_int(rng, 1_000, 10_000_000),
                    lam=rng.choice([5.0, 7.0, 9.0]), coding=coding, n_compact=c)
    if kind == "multi":
        return dict(kind=kind, tables=rng.randint(2, 16), n=_log_int(rng, 20_000, 2_000_000),
                    requests=rng.randint(3, 100), q_lo=1_000, q_hi=_log_int(rng, 20_000, 300_000),
                    lam=rng.choice([5.0, 7.0]), mix=rng.randint(1, 9999))
    if kind == "build":
        return dict(kind=kind, n=_log_int(rng, 1_000, 100_000_000), lam=rng.choice([5.0, 7.0, 8.0, 9.0]), P=2500,
                    coding=coding, bucket_fn=rng.choice(["optimized", "optimized", "optimized", "skew"]),
                    order=rng.choice(["random", "random", "serial"]))
    if kind == "wide":
        return dict(kind="build", n=_log_int(rng, 100_000, 10_000_000), lam=rng.choice([5.0, 7.0]),
                    P=rng.choice([1_000, 10_000, 20_000, 50_000, 100_000]), coding="rice", bucket_fn="optimized",
                    order="random")
    if kind == "dense":
        return dict(kind="build", n=_log_int(rng, 2_500, 400_000), lam=rng.choice([10.0, 11.0, 12.0]), P=2500,
                    coding=coding, bucket_fn="optimized", order="random")
    if kind == "strings":
        hi = rng.choice([16, 50, 90])
        a = rng.choice([(1, 1), (99, 100)])
        return dict(kind=kind, n=_log_int(rng, 5_000, 10_000_000), lam=rng.choice([5.0, 7.0]), coding=coding,
                    alpha_num=a[0], alpha_den=a[1], lo=10, hi=hi)
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(3, 512), median=_log_int(rng, 5_000, 50_000),
                    lam=rng.choice([5.0, 7.0]), mix=rng.randint(1, 9999))
    if kind == "load":
        return dict(kind=kind, n=_log_int(rng, 10_000, 10_000_000), q=_log_int(rng, 1_000, LOOKUPS),
                    lam=rng.choice([5.0, 7.0, 9.0]), coding=coding)
    return dict(kind=kind, tables=rng.randint(2, 8), n=_log_int(rng, 50_000, 1_000_000), queries=rng.randint(8, 80),
                q_lo=1_000, q_hi=_log_int(rng, 50_000, 1_000_000), builds=rng.randint(1, 8),
                median=_log_int(rng, 50_000, 500_000), lam=rng.choice([5.0, 7.0]), mix=rng.randint(1, 9999))


# --- inputs -------------------------------------------------------------------------------------

def _i64(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _keys(n, stream):
    """n distinct u64 keys spread over the whole range: a bijection of a counter (stream picks which)."""
    x = torch.arange(n, dtype=torch.int64, device="cuda")
    x += _i64(stream * 0xD1342543DE82EF95)
    for c in (0xD6E8FEB86659FD93, 0xA5CB9243F0AEF6D5):
        x ^= (x >> 32) & 0xFFFFFFFF
        x *= _i64(c)
    x ^= (x >> 29) & 0x7FFFFFFFF
    return x


def _serial(n, stream):
    """n consecutive ids."""
    return torch.arange(n, dtype=torch.int64, device="cuda") + _i64(stream * 0x2545F4914F6CDD1D) // 4


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _pick(keys, q, g):
    return keys[torch.randint(0, keys.numel(), (q,), generator=g, device="cuda")]


def _strings(n, lo, hi, seed):
    g = _gen(seed)
    lens = torch.randint(lo, hi + 1, (n,), generator=g, device="cuda")
    offs = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=offs[1:])
    chars = torch.tensor(list(b"abcdefghijklmnopqrstuvwxyz0123456789"), dtype=torch.uint8, device="cuda")
    total = int(offs[-1])
    data = torch.empty(total, dtype=torch.uint8, device="cuda")
    step = 1 << 26
    for a in range(0, total, step):
        b = min(total, a + step)
        data[a:b] = chars[torch.randint(0, 36, (b - a,), generator=g, device="cuda")]
    return data, offs


def _sizes(case, count):
    """Key counts of the case's tables (its "mix" picks them, the seed only the keys)."""
    rng = np.random.default_rng(case["mix"])
    x = rng.lognormal(mean=math.log(case["median"]), sigma=1.5, size=count)
    return [int(v) for v in np.clip(np.rint(x), 1_000, 2_000_000)]


def _requests(case, count):
    rng = np.random.default_rng(case["mix"] + 10_000)
    return [int(v) for v in np.rint(np.exp(rng.uniform(math.log(case["q_lo"]), math.log(case["q_hi"]), count)))]


def _params(case):
    return phobic.params(partition_size=case.get("P", 2500), lam=case["lam"], coding=case.get("coding", "rice"),
                         alpha=(case.get("alpha_num", 1), case.get("alpha_den", 1)),
                         n_compact=case.get("n_compact", 0), bucket_fn=case.get("bucket_fn", "optimized"))


def _split(buf, sizes):
    return list(torch.split(buf, sizes))


def prepare(case, seed):
    kind, prm, g = case["kind"], _params(case), _gen(seed)
    st = dict(case=case, prm=prm)
    if kind == "query":
        keys = _keys(case["n"], seed)
        st["h"] = phobic.build_u64(keys, prm)
        st["q"] = _pick(keys, case["q"], g)
        st["out"] = torch.empty_like(st["q"])
    elif kind == "multi":
        sets = [_keys(case["n"], seed * 1009 + t) for t in range(case["tables"])]
        tables = [phobic.build_u64(k, prm) for k in sets]
        ns = _requests(case, case["requests"])
        st["h"] = [tables[r % case["tables"]] for r in range(len(ns))]
        st["q"] = [_pick(sets[r % case["tables"]], n, g) for r, n in enumerate(ns)]
        st["buf"] = torch.empty(sum(ns), dtype=torch.int64, device="cuda")
        st["outs"] = _split(st["buf"], ns)
    elif kind == "build":
        st["keys"] = _serial(case["n"], seed) if case["order"] == "serial" else _keys(case["n"], seed)
    elif kind == "strings":
        st["data"], st["offs"] = _strings(case["n"], case["lo"], case["hi"], seed)
    elif kind == "batch":
        ns = _sizes(case, case["count"])
        st["all"] = _keys(sum(ns), seed)
        st["sets"] = phobic.BatchKeys(_split(st["all"], ns))
        st["buf"] = torch.empty(sum(ns), dtype=torch.int64, device="cuda")
        st["outs"] = _split(st["buf"], ns)
    elif kind == "load":
        keys = _keys(case["n"], seed)
        st["image"] = phobic.build_u64(keys, prm).serialize()
        st["q"] = _pick(keys, case["q"], g)
    elif kind == "serve":
        sets = [_keys(case["n"], seed * 1009 + t) for t in range(case["tables"])]
        ns = _requests(case, case["queries"])
        bs = _sizes(case, case["builds"])
        st["q"] = [_pick(sets[r % case["tables"]], n, g) for r, n in enumerate(ns)]
        st["new"] = [_keys(n, seed * 1009 + 500 + t) for t, n in enumerate(bs)]
        st["buf"] = torch.empty(sum(ns) + sum(bs), dtype=torch.int64, device="cuda")
        st["outs"] = _split(st["buf"], ns + bs)
        torch.cuda.current_stream().synchronize()  # the server works on streams of its own
        srv = phobic.Server(prm, budget_bytes=64 << 30, workers=4, max_query_batch=64, max_build_batch=8,
                            query_workers=1)
        ids = [srv.submit_build(k) for k in sets]
        _wait(srv, ids)
        st["srv"], st["ids"] = srv, ids
    return st


def _wait(srv, ids):
    left = set(ids)
    while left:
        for r in srv.poll(wait_ms=1000):
            if r["status"] != 0:
                raise RuntimeError("request failed: %r" % (r,))
            left.discard(r["request_id"])


# --- one pass -----------------------------------------------------------------------------------

def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "query":
        return st["h"].query_u64(st["q"], out=st["out"])
    if kind == "multi":
        phobic.query_multi_u64(st["h"], st["q"], st["outs"])
        return st["buf"]
    if kind == "build":
        h = phobic.build_u64(st["keys"], st["prm"])
        return {"pos": h.query_u64(st["keys"]), "bits": h.size_bits()}
    if kind == "strings":
        h = phobic.build_str(st["data"], st["offs"], st["prm"])
        return {"pos": h.query_str(st["data"], st["offs"]), "bits": h.size_bits()}
    if kind == "batch":
        hs = phobic.build_batch_u64(st["sets"], st["prm"])
        phobic.query_multi_u64(list(hs), st["sets"].tensors, st["outs"])
        return {"pos": st["buf"], "bits": sum(h.size_bits() for h in hs)}
    if kind == "load":
        h = phobic.deserialize(st["image"])
        return h.query_u64(st["q"])
    # serve: the queries arrive with the builds among them; every new table is queried once, then dropped
    srv, nq, nb = st["srv"], len(st["q"]), len(st["new"])
    every = max(1, nq // nb)
    ids, made = [], []
    for r, q in enumerate(st["q"]):
        ids.append(srv.submit_query(st["ids"][r % case["tables"]], q, st["outs"][r]))
        if r % every == 0 and len(made) < nb:
            made.append(srv.submit_build(st["new"][len(made)]))
    while len(made) < nb:
        made.append(srv.submit_build(st["new"][len(made)]))
    for t, m in enumerate(made):
        ids.append(srv.submit_query(m, st["new"][t], st["outs"][nq + t]))
    _wait(srv, ids + made)
    for m in made:
        srv.release(m)
    return st["buf"]


# --- the least a pass moves ---------------------------------------------------------------------

def _image(n):
    return 0.25 * n  # about two bits per key


def work(case):
    kind = case["kind"]
    if kind == "query":  # a key and a position per lookup, and the part of the table that they touch
        return {"bytes": 16 * case["q"] + min(_image(case["n"]), 16 * case["q"]), "flops": 0}
    if kind == "multi":
        return {"bytes": 16 * sum(_requests(case, case["requests"])), "flops": 0}
    if kind == "build":
        return {"bytes": 16 * case["n"] + 2 * _image(case["n"]), "flops": 0}
    if kind == "strings":
        return {"bytes": (16 + (case["lo"] + case["hi"]) / 2) * case["n"] + 2 * _image(case["n"]), "flops": 0}
    if kind == "batch":
        n = sum(_sizes(case, case["count"]))
        return {"bytes": 16 * n + 2 * _image(n), "flops": 0}
    if kind == "load":
        return {"bytes": _image(case["n"]) + 16 * case["q"], "flops": 0}
    n = sum(_sizes(case, case["builds"]))
    return {"bytes": 16 * sum(_requests(case, case["queries"])) + 16 * n + 2 * _image(n), "flops": 0}
