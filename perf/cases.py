"""The work that the performance of this library is judged by.

listed() names the cases, draw() gives more of the same ranges, prepare() makes what a user's
program holds before the call (handles, inputs, buffers), run() makes one pass through the
public API, work() says what a pass cannot do without, and exact() what it has to return.

Every result that run() returns is determined by the inputs: latencies, waiting times and
the high-water marks that depend on the schedule (most holders seen, most values queued)
are left out.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1110_4623_amd as sp
import sp_inputs

WAVES_PER_CU, CUS = 32, 256  # what a barrier's co-residency allows


def listed():
    return [
        # Barriers.  A small solver's grid, one wavefront per workgroup: few workgroups that
        # meet often.
        {"name": "barrier 16 x 64", "path": "barrier", "nwg": 16, "lanes": 64, "rounds": 1000,
         "coherent": False},
        # Iterations of a mid-size kernel whose exchanged words are accessed coherently (the
        # paper's volatile data), an odd workgroup size and count.
        {"name": "barrier 1000 x 192 coherent", "path": "barrier", "nwg": 1000, "lanes": 192,
         "rounds": 2000, "coherent": True},
        # The full GPU, plain data: a persistent kernel's global synchronization.
        {"name": "barrier 2048 x 256", "path": "barrier", "nwg": 2048, "lanes": 256,
         "rounds": 10_000, "coherent": False},
        # Mutexes.  The smallest call: a handful of updates of one-word records.
        {"name": "mutex 24 on 16 locks", "path": "mutex", "nwg": 24, "lanes": 64, "locks": 16,
         "words": 1, "total": 480, "delay": 100, "coherent": False},
        # One hot lock that every resident workgroup wants.
        {"name": "mutex 2048 on 1 lock", "path": "mutex", "nwg": 2048, "lanes": 256, "locks": 1,
         "words": 16, "total": 1 << 16, "delay": 1000, "coherent": False},
        # A hash table's worth of locks over larger records.
        {"name": "mutex 2048 on 256 locks", "path": "mutex", "nwg": 2048, "lanes": 256,
         "locks": 256, "words": 256, "total": 1 << 19, "delay": 1000, "coherent": False},
        # Semaphores.  A pool of 32 resources that a full GPU competes for.
        {"name": "semaphore K 32, 2048", "path": "semaphore", "nwg": 2048, "lanes": 256, "K": 32,
         "total": 1 << 18, "hold": 2000, "data": False, "coherent": False},
        # A small pool whose holders update what it guards, an odd number of contenders.
        {"name": "semaphore K 4, 257, data", "path": "semaphore", "nwg": 257, "lanes": 128,
         "K": 4, "total": 1 << 14, "hold": 500, "data": True, "coherent": False},
        # A producer/consumer ring on a mutex and two condition variables.
        {"name": "ring 96 to 160", "path": "condition", "mutex": "ticket", "nwg": 256,
         "producers": 96, "lanes": 64, "capacity": 64, "items": 10_000},
        # The persistent queue at a high arrival rate.
        {"name": "serve 10000 at 1e6", "path": "serving", "nwg": 1024, "n": 10_000, "rate": 1e6},
        # Memory-system microbenchmarks: distributed atomics over a million words, and the
        # streaming read.
        {"name": "atomics 2^20 words", "path": "atomics", "op": "add", "mode": "per_lane",
         "nwg": 2048, "lanes": 256, "T": 1 << 20, "stride": 64, "ops": 16},
        {"name": "stream 1 GiB", "path": "stream", "bytes": 1 << 30},
    ]


def _log_int(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _grid(rng, most):
    """Workgroups (up to `most`) and lanes of a grid that is resident at once."""
    lanes = 64 * rng.choice([1, 1, 2, 3, 4, 4, 5, 8, 16])
    return _log_int(rng, 2, min(most, CUS * (WAVES_PER_CU // (lanes // 64)))), lanes


def draw(rng):
    path = rng.choice([c["path"] for c in listed()])
    c = {"path": path}
    if path == "barrier":
        c["nwg"], c["lanes"] = _grid(rng, 2048)
        c["rounds"] = _log_int(rng, 10, 5000)
        c["coherent"] = rng.random() < 0.33
    elif path == "mutex":
        c["nwg"], c["lanes"] = _grid(rng, 2048)
        c["locks"] = _log_int(rng, 1, 256)
        c["words"] = _log_int(rng, 1, 256)
        c["total"] = _log_int(rng, 200, min(16_000 * min(c["locks"], c["nwg"]), 1 << 18))
        c["delay"] = rng.randint(0, 1000)
        c["coherent"] = rng.random() < 0.25
    elif path == "semaphore":
        c["nwg"], c["lanes"] = _grid(rng, 2048)
        c["K"] = _log_int(rng, 1, 256)
        c["total"] = _log_int(rng, 200, min(8000 * min(c["K"], c["nwg"]), 1 << 18))
        c["hold"] = rng.randint(0, 2000)
        c["data"] = rng.random() < 0.5
        c["coherent"] = rng.random() < 0.25
    elif path == "condition":
        c["mutex"] = rng.choice(["ticket", "array", "cohort"])
        c["nwg"] = _log_int(rng, 2, 512)
        c["producers"] = rng.randint(1, c["nwg"] - 1)
        c["lanes"] = 64 * rng.choice([1, 2, 4])
        c["capacity"] = _log_int(rng, 4, 4096)
        c["items"] = _log_int(rng, 200, 10_000)
    elif path == "serving":
        c["nwg"] = _log_int(rng, 64, 1024)
        c["rate"] = float(_log_int(rng, 100_000, 1_000_000))
        c["n"] = _log_int(rng, 500, int(0.02 * c["rate"]))
    elif path == "atomics":
        c["op"] = rng.choice(["add", "cas", "ld", "st"])
        c["mode"] = rng.choice(["per_lane", "wave_leader"])
        c["nwg"] = _log_int(rng, 1, 2048)
        c["lanes"] = 64 * rng.choice([1, 2, 4])
        # a compare-and-swap loop's retries grow with the square of the contenders of a word
        c["T"] = _log_int(rng, 65_536 if c["op"] == "cas" else 32, 1 << 20)
        c["stride"] = rng.choice([4, 64, 128])
        c["ops"] = _log_int(rng, 1, 16)
    else:
        c["bytes"] = 16 * _log_int(rng, 1 << 14, 1 << 26)
    return c


# ---- inputs ---------------------------------------------------------------------------

_CTX = None


def _ctx():
    global _CTX
    if _CTX is None:
        _CTX = sp.Context(0)
    return _CTX


def _u32(seed):
    return (seed * 2654435761 + 12345) & 0xFFFFFFFF


def _total(c, seed):
    """A program's operation count is not a round number: it changes with the input."""
    return c["total"] - seed % (1 + c["total"] // 64)


def _rate_table(c, seed):
    return sp_inputs.request_table(c["n"], c["rate"], seed)


def _words(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-(1 << 31), 1 << 31, (c["bytes"] // 4,), dtype=torch.int32,
                         device="cuda", generator=g)


def prepare(case, seed):
    ctx, c = _ctx(), case
    s = {"ctx": ctx, "case": c, "seed": _u32(seed)}
    if c["path"] == "barrier":
        s["barrier"] = sp.Barrier(ctx, "default", c["nwg"], coherent_cs=int(c["coherent"]))
    elif c["path"] == "mutex":
        s["mutex"] = sp.Mutex(ctx, "default", c["locks"], c["words"],
                              coherent_cs=int(c["coherent"]))
        s["total"] = _total(c, seed)
    elif c["path"] == "semaphore":
        s["sem"] = sp.Semaphore(ctx, "default", c["K"], coherent_cs=int(c["coherent"]))
        s["total"] = _total(c, seed)
    elif c["path"] == "serving":
        s["requests"] = _rate_table(c, seed)
    elif c["path"] == "atomics":
        s["perm"] = ctx.upload(sp_inputs.permutation(c["T"], seed))
        s["buf"] = ctx.zeros(c["T"] * c["stride"] // 4)
    elif c["path"] == "stream":
        s["words"] = _words(c, seed)
    return s


def run(s):
    c, ctx, seed = s["case"], s["ctx"], s["seed"]
    if c["path"] == "barrier":
        checksums, _ = s["barrier"].run_hash(c["lanes"], c["rounds"], seed)
        return checksums
    if c["path"] == "mutex":
        words, _, _ = s["mutex"].run(c["nwg"], c["lanes"], s["total"], c["delay"], seed)
        return words
    if c["path"] == "semaphore":
        r = s["sem"].run(c["nwg"], c["lanes"], s["total"], c["hold"], seed, track=True,
                         data=c["data"])
        # which slot of the pool an admission took is not unique: only their sum is
        held = int(r["data"].sum(dtype=np.uint64)) if c["data"] else 0
        return {"chk": r["chk"], "admissions": r["state"][3], "count": r["count"],
                "inside": r["occ"], "unserved": r["unserved"], "held": held,
                "over": int(r["maxocc"] > c["K"])}
    if c["path"] == "condition":
        r = sp.bounded_buffer(ctx, c["mutex"], c["nwg"], c["producers"], c["capacity"],
                              c["items"], seed, lanes=c["lanes"])
        return {k: r[k] for k in ("xor", "sum", "taken", "put", "left")}
    if c["path"] == "serving":
        out, _, r = sp.serve(ctx, s["requests"], nwg=c["nwg"], seed=seed)
        return {"out": out, "completed": r["completed"], "issued": r["units_issued"],
                "released": r["units_released"]}
    if c["path"] == "atomics":
        finals, total, _ = sp.bench_atomic(ctx, c["op"], c["nwg"], c["lanes"], c["T"],
                                           c["stride"], c["mode"], c["ops"], seed, s["perm"],
                                           s["buf"])
        return {"finals": finals, "sum": total}
    total, _ = sp.stream_read(ctx, s["words"], c["bytes"])
    return total


# ---- what a pass cannot do without -------------------------------------------------------

def _issuers(c):
    return c["nwg"] * (c["lanes"] if c["mode"] == "per_lane" else c["lanes"] // 64)


def work(case):
    """Bytes: every exchanged or guarded word read and written once per operation, inputs
    and outputs once.  flops: integer operations of the workload's hashes (nine each)."""
    c = case
    if c["path"] == "barrier":
        n = c["nwg"] * c["rounds"]
        return {"bytes": 8 * n + 4 * c["nwg"], "flops": 9 * n}
    if c["path"] == "mutex":
        return {"bytes": 8 * c["words"] * c["total"] + 4 * c["words"] * c["locks"],
                "flops": c["words"] * c["total"]}
    if c["path"] == "semaphore":
        return {"bytes": (16 if c["data"] else 8) * c["total"] + 4 * c["nwg"],
                "flops": 9 * c["total"]}
    if c["path"] == "condition":
        return {"bytes": 8 * c["items"], "flops": 9 * c["items"]}
    if c["path"] == "serving":
        # a lognormal(5, 1.5) chain has about 440 steps on average
        return {"bytes": 24 * c["n"], "flops": 9 * 440 * c["n"]}
    if c["path"] == "atomics":
        n = _issuers(c) * c["ops"]
        return {"bytes": (4 if c["op"] in ("ld", "st") else 8) * n + 8 * c["T"], "flops": n}
    return {"bytes": c["bytes"] + 8, "flops": c["bytes"] // 4}


# ---- what a pass has to return -----------------------------------------------------------

def _sm32(x):
    with np.errstate(over="ignore"):  # arithmetic modulo 2^32
        z = np.asarray(x, dtype=np.uint32) + np.uint32(0x9E3779B9)
        z = (z ^ (z >> np.uint32(16))) * np.uint32(0x85EBCA6B)
        z = (z ^ (z >> np.uint32(13))) * np.uint32(0xC2B2AE35)
        return z ^ (z >> np.uint32(16))


def _shares(total, n):
    return [total // n + (w < total % n) for w in range(n)]


def _hashes(seed, w, n):
    return _sm32(np.uint32((seed ^ (w << 16)) & 0xFFFFFFFF) ^ np.arange(n, dtype=np.uint32))


def exact(case, seed):
    c, s = case, _u32(seed)
    if c["path"] == "barrier":
        b = np.arange(c["nwg"], dtype=np.uint32)
        chk = np.zeros(c["nwg"], dtype=np.uint32)
        for r in range(c["rounds"]):
            v = _sm32(np.uint32(s) ^ (b << np.uint32(16)) ^ np.uint32(r))
            chk ^= np.roll(v, -(r % c["nwg"]))
        return chk
    if c["path"] == "mutex":
        counts = np.zeros(c["locks"], dtype=np.int64)
        key = _sm32(np.uint32(s ^ 1))
        for w, n in enumerate(_shares(_total(c, seed), c["nwg"])):
            k = _sm32(_sm32(key ^ np.uint32(w)) ^ np.arange(n, dtype=np.uint32))
            counts += np.bincount(k % np.uint32(c["locks"]), minlength=c["locks"])
        return np.repeat(counts[:, None], c["words"], axis=1).astype(np.uint32)
    if c["path"] == "semaphore":
        total = _total(c, seed)
        chk = [np.bitwise_xor.reduce(_hashes(s, w, n), initial=np.uint32(0))
               for w, n in enumerate(_shares(total, c["nwg"]))]
        return {"chk": np.array(chk, dtype=np.uint32), "admissions": total, "count": 0,
                "inside": 0, "unserved": 0, "held": total if c["data"] else 0, "over": 0}
    if c["path"] == "condition":
        v = np.concatenate([_hashes(s, w, n)
                            for w, n in enumerate(_shares(c["items"], c["producers"]))])
        return {"xor": int(np.bitwise_xor.reduce(v)), "sum": int(v.sum(dtype=np.uint64)),
                "taken": c["items"], "put": c["items"], "left": 0}
    if c["path"] == "serving":
        t = _rate_table(c, seed)
        h = np.uint32(s) ^ np.arange(c["n"], dtype=np.uint32)
        order = np.argsort(-t["L"].astype(np.int64))
        h, L = h[order], t["L"][order].astype(np.int64)
        live = len(L)
        for i in range(int(L[0])):
            while L[live - 1] <= i:
                live -= 1
            h[:live] = _sm32(h[:live])
        out = np.empty(c["n"], dtype=np.uint32)
        out[order] = h
        units = int(((t["nbytes"] + 65535) // 65536).sum())
        return {"out": out, "completed": c["n"], "issued": units, "released": units}
    if c["path"] == "atomics":
        T = c["T"]
        first = np.bincount(np.arange(_issuers(c)) % T, minlength=T)
        hits = np.zeros(T, dtype=np.int64)
        for i in range(c["ops"]):
            hits += np.roll(first, i)
        at = sp_inputs.permutation(T, seed)
        seen = np.empty(T, dtype=np.int64)
        seen[at] = hits
        value = _sm32(np.uint32(s) ^ np.arange(T, dtype=np.uint32))
        if c["op"] == "ld":
            return {"finals": value, "sum": int((seen * value.astype(np.int64)).sum())}
        if c["op"] == "st":
            return {"finals": np.where(seen > 0, value, 0).astype(np.uint32), "sum": 0}
        return {"finals": seen.astype(np.uint32), "sum": int((seen * (seen - 1) // 2).sum())}
    return int((_words(c, seed).to(torch.int64) & 0xFFFFFFFF).sum())
