"""Performance cases of liblabs: what a user's program has the library do.

Every case is one call of the public Python front end (``Labs`` and
``Server``) at a size of the workload recipes in
``paper_2504_00987_amd/inputs.py`` or of the benchmark, or, when drawn, at a
size of the same ranges.  ``prepare`` makes the inputs from the seed,
``run`` is one pass, ``work`` what a pass cannot do without.

Searches (walks, memetic generations, served solves) are sequences of integer
decisions, defined bit for bit by their seed: they have no value of their own
in 64 bits.  Energies and d(S) do (``exact``).
"""
import math
import random
import time

import numpy as np
import torch

from paper_2504_00987_amd import inputs as I
from paper_2504_00987_amd.labs import Labs, Server


def listed():
    return [
        # a first call, a test, one interactive query: launch and latency bound
        dict(name="walks_few", kind="walks", walks=64, lo=64, hi=64, mult=2, starts=False),
        # short sequences, enough walks to fill the device
        dict(name="walks_n32", kind="walks", walks=16384, lo=32, hi=32, mult=4, starts=False),
        # the default benchmark workload
        dict(name="walks_n64", kind="walks", walks=4096, lo=64, hi=64, mult=4, starts=False),
        # a batch of every length in the range of the paper's record searches
        dict(name="walks_uneven", kind="walks", walks=8192, lo=48, hi=120, mult=3, starts=False),
        # improving sequences the caller already has (its own starts)
        dict(name="walks_n120_starts", kind="walks", walks=4096, lo=120, hi=120, mult=4,
             starts=True),
        # long sequences of mixed lengths: the largest walk batch
        dict(name="walks_long_uneven", kind="walks", walks=4096, lo=129, hi=256, mult=4,
             starts=False),
        # the memetic search itself (Alg. 1): one replica per compute unit
        dict(name="memetic_n120", kind="memetic", pops=256, lo=120, hi=120, gens=64, children=1),
        # its batched-generation form
        dict(name="memetic_n120_children8", kind="memetic", pops=256, lo=120, hi=120, gens=16,
             children=8),
        # scoring a large set of sequences of mixed lengths
        dict(name="energies", kind="energies", rows=262144, lo=20, hi=128),
        # analysis of results: deviation from skew-symmetry (App. A)
        dict(name="skew_deviation", kind="skew", rows=4096, lo=120, hi=120),
        # one small-N time-to-solution run: the exhaustive minimum, then the search until it is hit
        dict(name="solution_n33", kind="solution", n=33),
        # the serving loop: a burst of solve requests of mixed lengths
        dict(name="serving_burst", kind="serving", requests=128, lo=32, hi=128, pops=16, gens=50),
    ]


def _spread(rng, lo, hi):
    """A whole number in [lo, hi], uniform over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw(rng):
    kind = rng.choice(["walks", "walks", "walks", "memetic", "memetic", "energies", "skew",
                       "solution", "serving"])
    if kind == "walks":
        lo = _spread(rng, 3, 256)
        lo, hi = rng.choice([(lo, lo), (lo, rng.randint(lo, 256))])
        return dict(kind=kind, walks=_spread(rng, 1, 16384), lo=lo, hi=hi,
                    mult=rng.randint(1, 4), starts=rng.random() < 0.3)
    if kind == "memetic":
        lo = _spread(rng, 12, 200)
        lo, hi = rng.choice([(lo, lo), (lo, rng.randint(lo, 200))])
        return dict(kind=kind, pops=_spread(rng, 1, 1024), lo=lo, hi=hi,
                    gens=_spread(rng, 4, 64), children=rng.choice([1, 1, 2, 4, 8]))
    if kind == "energies":
        lo = rng.randint(3, 256)
        return dict(kind=kind, rows=_spread(rng, 1, 262144), lo=lo, hi=rng.randint(lo, 256))
    if kind == "skew":
        lo = rng.randint(9, 160)
        lo, hi = rng.choice([(lo, lo), (lo, rng.randint(lo, 160))])
        return dict(kind=kind, rows=_spread(rng, 1, 4096), lo=lo, hi=hi)
    if kind == "solution":
        return dict(kind=kind, n=rng.randint(16, 33))
    lo = rng.randint(24, 128)
    return dict(kind=kind, requests=_spread(rng, 1, 128), lo=lo, hi=rng.randint(lo, 128), pops=16,
                gens=_spread(rng, 10, 50))


def draw(rng):
    most = {}
    for c in listed():
        w = work(c)
        most[c["kind"]] = max(most.get(c["kind"], 0.0), w["flops"])
    while True:
        c = _draw(rng)
        if work(c)["flops"] <= most[c["kind"]]:
            return c


def _lengths(case, count, seed):
    """None for one length, else int32 lengths uniform in lo..hi."""
    if case["lo"] == case["hi"]:
        return None
    return I.uneven_lengths(count, case["lo"], case["hi"], seed)


def _rows(case, count, seed):
    """(int8 +-1 rows, zero past their length; lengths or None), in host memory."""
    ns = _lengths(case, count, seed)
    if ns is None:
        return I.random_pm1(count, case["hi"], case["hi"], seed + 1), None
    rows = I.random_pm1(count, case["hi"], case["hi"], seed + 1)
    rows[np.arange(case["hi"])[None, :] >= ns[:, None]] = 0
    return rows, ns


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case, "seed": seed, "lb": Labs(0)}
    if kind == "walks":
        st["rules"] = I.rules_tabu(case["mult"])
        st["starts"] = None
        if case["starts"]:
            rows, st["ns"] = _rows(case, case["walks"], seed)
            st["starts"] = torch.from_numpy(rows).cuda()
        else:
            st["ns"] = _lengths(case, case["walks"], seed)
    elif kind == "memetic":
        st["ns"] = _lengths(case, case["pops"], seed)
    elif kind in ("energies", "skew"):
        rows, ns = _rows(case, case["rows"], seed)
        st["rows"] = torch.from_numpy(rows).cuda()
        st["ns"] = None if ns is None else torch.from_numpy(ns).cuda()
    elif kind == "serving":
        ns = np.random.default_rng(seed).integers(case["lo"], case["hi"] + 1,
                                                  size=case["requests"])
        st["reqs"] = [(int(n), seed * 1000003 + i) for i, n in enumerate(ns)]
        st["server"] = Server(st["lb"], 100, I.RULES_MEMETIC, 8192, chunk=25)
    return st


def run(st):
    case, lb = st["case"], st["lb"]
    uniform = case["hi"] if case.get("lo", 0) == case.get("hi", -1) else 0
    stride = max(128, case.get("hi", 0))  # rows of the search results
    if st["kind"] == "walks":
        r = lb.tabu_batch(st["rules"], case["walks"], st["seed"], ns=st["ns"], n_uniform=uniform,
                          starts=st["starts"], out_stride=stride)
        return {"best_seq": r.best_seq, "best_e": r.best_e, "final_e": r.final_e}
    if st["kind"] == "memetic":
        r = lb.memetic_run(100, I.RULES_MEMETIC, case["gens"], case["pops"], st["seed"],
                           ns=st["ns"], n_uniform=uniform, out_stride=stride,
                           children=case["children"])
        return {"best_seq": r.best_seq, "best_e": r.best_e, "hit_gen": r.hit_gen,
                "gens_done": r.gens_done}
    if st["kind"] == "energies":
        return lb.energy_batch(st["rows"], st["ns"], uniform)
    if st["kind"] == "skew":
        return lb.skew_deviation(st["rows"], st["ns"], uniform)
    if st["kind"] == "solution":
        e, count, seq = lb.bruteforce_min(case["n"])
        r = lb.memetic_run(100, I.RULES_PAPER_LITERAL, 10**6, 64, st["seed"],
                           n_uniform=case["n"], chunk=16, target=e, stop_all=1)
        return {"min_e": e, "count": count, "argmin": seq, "best_seq": r.best_seq,
                "best_e": r.best_e, "hit_gen": r.hit_gen, "gens_done": r.gens_done}
    # a client that submits its requests and collects the answers in order
    srv = st["server"]
    ids = [srv.submit(n, s, case["pops"], case["gens"]) for n, s in st["reqs"]]
    seqs = np.zeros((len(ids), case["hi"]), dtype=np.int8)
    best = np.zeros(len(ids), dtype=np.int32)
    for i, (rid, (n, _)) in enumerate(zip(ids, st["reqs"])):
        while (got := srv.poll(rid, n)) is None:
            time.sleep(1e-4)
        seqs[i, :n], best[i] = got[0], got[1]
    return {"best_seq": seqs, "best_e": best}


def _mean_n(case, power):
    lo, hi = case["lo"], case["hi"]
    return sum(n ** power for n in range(lo, hi + 1)) / (hi - lo + 1)


def work(case):
    """Bytes: inputs once, outputs once.  Operations, one per number changed
    or compared: a step of a walk changes N neighbour scores and the N
    correlations they are made of, and compares the scores; a start takes
    N^2 / 2 products; d(S) at least one count per rotation (odd N) or per
    rotation and deletion (even N); the exhaustive minimum what the published
    branch and bound takes (N 1.73^N, Packebusch and Mertens 2016)."""
    kind = case["kind"]
    if kind == "solution":
        return {"bytes": case["n"] + 12 + 64 * (128 + 20), "flops": case["n"] * 1.73 ** case["n"]}
    n1, n2 = _mean_n(case, 1), _mean_n(case, 2)
    if kind == "walks":
        stride = max(128, case["hi"])
        return {"bytes": case["walks"] * (stride + 8 + (n1 if case["starts"] else 0)
                                          + (4 if case["lo"] < case["hi"] else 0)),
                "flops": case["walks"] * (case["mult"] * 4 * n2 + n2)}
    if kind == "memetic":
        # a walk of N steps on average per child
        return {"bytes": case["pops"] * (max(128, case["hi"]) + 20),
                "flops": case["pops"] * (case["gens"] * case["children"] * 5 * n2 + 100 * n2 / 2)}
    if kind == "serving":
        reps = case["requests"] * case["pops"]
        return {"bytes": case["requests"] * (n1 + 4),
                "flops": reps * (case["gens"] * 5 * n2 + 100 * n2 / 2)}
    if kind == "energies":
        words = math.ceil(case["hi"] / 32)
        return {"bytes": case["rows"] * (n1 + 4 + (4 if case["lo"] < case["hi"] else 0)),
                "flops": case["rows"] * n1 * (3 * words / 2 + 2)}
    odd = [n for n in range(case["lo"], case["hi"] + 1) if n & 1]
    even = [n for n in range(case["lo"], case["hi"] + 1) if not n & 1]
    counts = (sum(n * math.ceil(n / 32) for n in odd) + sum(n * n for n in even))
    return {"bytes": case["rows"] * (n1 + 4 + (4 if case["lo"] < case["hi"] else 0)),
            "flops": case["rows"] * counts / (len(odd) + len(even))}


def _exact_energies(rows, ns):
    """Eq. 1-2: the squares of the aperiodic autocorrelations, lag by lag."""
    r = torch.from_numpy(rows).to(torch.int64)  # zeros past a row's length add nothing
    e = torch.zeros(r.shape[0], dtype=torch.int64)
    for k in range(1, r.shape[1]):
        c = (r[:, :-k] * r[:, k:]).sum(1)
        e += c * c
    return e


def _exact_skew(row):
    """d(S) of one row: the least number of broken pairs t_{c+i} != (-1)^i
    t_{c-i} over rotations (odd N), or rotations and one deletion (even N)."""
    n = len(row)
    rot = row[(np.arange(n)[:, None] + np.arange(n)[None, :]) % n]
    if n % 2 == 0:  # every rotation without its element q, all q
        keep = np.array([[i for i in range(n) if i != q] for q in range(n)])
        rot = rot[:, keep].reshape(n * n, n - 1)
    c = (rot.shape[1] - 1) // 2
    i = np.arange(1, c + 1)
    sign = np.where(i % 2 == 1, -1, 1)
    return int((rot[:, c + i] != sign * rot[:, c - i]).sum(1).min())


def exact(case, seed):
    if case["kind"] == "energies":
        rows, ns = _rows(case, case["rows"], seed)
        if rows.size * rows.shape[1] > 6e9:
            return None
        return _exact_energies(rows, ns)
    if case["kind"] == "skew":
        rows, ns = _rows(case, case["rows"], seed)
        if rows.shape[0] * case["hi"] ** 3 > 2e9:
            return None
        lens = [case["hi"]] * len(rows) if ns is None else ns
        return torch.tensor([_exact_skew(r[:n].astype(np.int64)) for r, n in zip(rows, lens)])
    return None
