"""Joins whose speed matters, from the smallest call to the largest, for timing one build of the library against another.

``listed()`` names the cases, ``draw()`` gives others of the same ranges,
``prepare()`` makes what a program has in device memory before the call,
``run()`` is one pass through the binding, ``work()`` the bytes the operation
cannot do without and ``exact()`` its result by plain torch.

A case is one of four forms:
  join         one ``hj_join`` of R and S
  probe        one ``hj_probe`` of a table kept over R
  build_probe  ``hj_build`` over R, then one ``hj_probe`` by S
  batch        one run of a plan over many joins of uneven sizes
"""
from __future__ import annotations

import dataclasses
import math

import torch

import paper_1307_1955_amd.hj as hj
from paper_1307_1955_amd import gen
from paper_1307_1955_amd.gen import device as dgen

BASE = {
    "form": "join", "algo": "auto", "passes": 2, "b1": 6, "b2": 6, "hash": "identity", "one_pass": True,
    "n_r": 0, "n_s": 0,
    "domain": 0,      # S keys uniform over 1..domain
    "r_dup": 1,       # rows of R per key: 1 = a permutation of 1..n_r, else uniform over 1..n_r / r_dup
    "skew": 0.0,      # share of R on one key (the skewed sets of Section 5.1)
    "zipf": 0.0,      # theta of a Zipf-distributed S (0: uniform)
    "shift": 0,       # rows the rid columns start past a 16-byte boundary
    "jobs": 0, "r_min": 0, "r_max": 0, "spec_seed": 0,
}


def case(**kw):
    return {**BASE, **kw}


def listed():
    return [
        # the smallest joins of a served or batched load: R is one LDS table, latency and launches are all there is
        case(name="small_1k_3k", n_r=1024, n_s=3072, domain=2048),
        # a small dimension table against a few hundred thousand rows: one partitioning pass, launch-bound
        case(name="small_64k_256k", n_r=65536, n_s=262144, domain=131072),
        # 1M x 1M, every S tuple matching once (the check workload of the simple join, planned by the library)
        case(name="mid_1m_1m", n_r=1 << 20, n_s=1 << 20, domain=1 << 20),
        # the headline: 16M x 16M, two passes of 6 bits, half of S matching
        case(name="phj_16m_16m", algo="phj", n_r=1 << 24, n_s=1 << 24, domain=1 << 25),
        # the library's default parameters (two-pass output) on odd sizes, duplicate keys, the paper's hash
        # and rid columns at another alignment than the key columns
        case(name="phj_ragged_dup", algo="phj", one_pass=False, hash="murmur2", n_r=10000019, n_s=12345677,
             r_dup=2, domain=20000038, shift=1),
        # the simple hash join at the headline's size
        case(name="shj_16m_16m", algo="shj", n_r=1 << 24, n_s=1 << 24, domain=1 << 25),
        # a simple join's table built and probed as two calls, two-pass output
        case(name="shj_build_probe", form="build_probe", algo="shj", one_pass=False, n_r=300007, n_s=1200011,
             domain=400009),
        # a partitioned table kept in memory and probed by a fact table
        case(name="probe_4m_16m", form="probe", n_r=1 << 22, n_s=1 << 24, domain=1 << 23),
        # Zipf-skewed probes: 16M x 64M, theta 1
        case(name="zipf_16m_64m", n_r=1 << 24, n_s=1 << 26, domain=1 << 24, zipf=1.0),
        # skewed build side: a tenth of R on one key
        case(name="skew_1m_16m", n_r=1 << 20, n_s=1 << 24, domain=1 << 21, skew=0.1),
        # many independent joins in one captured plan
        case(name="batch_256", form="batch", jobs=256, r_min=1024, r_max=1 << 20, spec_seed=4),
        # the largest: more partitions than a counted second pass takes
        case(name="large_128m_256m", n_r=1 << 27, n_s=1 << 28, domain=1 << 28),
    ]


def draw(rng):
    def log(lo, hi):
        n = int(round(lo * math.exp(rng.random() * math.log(hi / lo))))
        return n | 1 if rng.random() < 0.5 else n

    if rng.random() < 0.08:
        return case(form="batch", jobs=rng.randint(24, 256), r_min=1024, r_max=log(1 << 16, 1 << 20),
                    spec_seed=rng.randrange(1 << 20))
    form = rng.choice(["join", "join", "join", "probe", "build_probe"])
    algo = rng.choice(["auto", "auto", "phj", "phj", "shj"])
    c = case(form=form, algo=algo, one_pass=rng.random() < 0.65, hash=rng.choice(["identity", "identity", "murmur2"]),
             shift=rng.choice([0, 0, 0, 1, 2, 3]))
    n_r = log(1 << 10, 1 << (24 if algo == "shj" else 26))
    n_s = min(log(n_r, 16 * n_r), 1 << (25 if algo == "shj" else 27))
    domain = max(n_r, int(n_r / rng.uniform(0.25, 1.0)))
    if algo == "phj":  # partitions of 1K to 4K rows of R, as the planner would consider
        bits = max(2, min(16, math.ceil(math.log2(max(2.0, n_r / 4096))) + rng.randint(0, 2)))
        if bits <= 10 and rng.random() < 0.5:
            c.update(passes=1, b1=bits, b2=0)
        else:
            c.update(passes=2, b1=(bits + 1) // 2, b2=bits // 2)
    kind = rng.random()
    if kind < 0.12:
        c["r_dup"] = rng.randint(2, 8)
    elif kind < 0.22 and algo != "shj":
        n_r = min(n_r, 1 << 22)
        n_s = max(n_r, min(n_s, 16 * n_r))
        c["skew"] = rng.choice([0.01, 0.1, 0.25])
        domain = 2 * n_r
    elif kind < 0.32:
        n_r = min(n_r, 1 << 22)
        n_s = max(n_r, min(n_s, 16 * n_r))
        c["zipf"] = rng.choice([0.5, 1.0])
        domain = n_r
    c.update(n_r=n_r, n_s=n_s, domain=domain)
    return c


def params_of(c):
    bits = (c["b1"], c["b2"]) if c["algo"] == "phj" else (6, 6)
    return hj.params(c["algo"], c["passes"], bits, hash=c["hash"], one_pass=c["one_pass"])


def shifted_rows(n, shift):
    return dgen.rows(n + shift)[shift:] if shift else dgen.rows(n)


def relations(c, seed):
    n_r, n_s = c["n_r"], c["n_s"]
    if c["r_dup"] > 1:
        rk = dgen.uniform_keys(seed, gen.STREAM_R_KEYS, n_r, max(1, n_r // c["r_dup"]))
    elif c["skew"]:
        rk = dgen.skewed_r(seed, n_r, 1, c["domain"], c["skew"])[0]
    else:
        rk = dgen.perm_keys(seed, gen.STREAM_R_KEYS, n_r)
    if c["zipf"]:
        cdf = torch.from_numpy(gen.zipf_cdf(n_r, c["zipf"])).cuda()
        sk = dgen.zipf_keys(seed, gen.STREAM_S_KEYS, n_s, cdf)
    else:
        sk = dgen.uniform_keys(seed, gen.STREAM_S_KEYS, n_s, c["domain"])
    return rk, shifted_rows(n_r, c["shift"]), sk, shifted_rows(n_s, c["shift"])


def job_specs(c, seed):
    return [dataclasses.replace(s, seed=seed) for s in gen.batch_specs(c["spec_seed"], c["jobs"], c["r_min"], c["r_max"])]


def expected_pairs(c):
    """Mean number of pairs."""
    if c["form"] == "batch":
        return sum(s.n_s * s.n_r / s.s_domain for s in job_specs(c, 0))
    return c["n_s"] if c["zipf"] else c["n_s"] * c["n_r"] / c["domain"]


def room(c):
    """Length of the result columns: every S tuple of a batch job (unique R keys), else room for half again the mean
    number of pairs past one for every S tuple, which a seed stays well within."""
    return sum(s.n_s for s in job_specs(c, 0)) if c["form"] == "batch" else c["n_s"] + int(1.5 * expected_pairs(c))


def columns(n):
    return torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")


def prepare(c, seed):
    if c["form"] == "batch":
        specs = job_specs(c, seed)
        rows = dgen.rows(max(max(s.n_r, s.n_s) for s in specs))
        out_r, out_s = columns(room(c))
        jobs, at = [], 0
        for s in specs:  # unique R keys: at most one pair per S tuple
            jobs.append((dgen.perm_keys(seed, s.r_stream, s.n_r), rows[: s.n_r],
                         dgen.uniform_keys(seed, s.s_stream, s.n_s, s.s_domain), rows[: s.n_s],
                         out_r[at: at + s.n_s], out_s[at: at + s.n_s]))
            at += s.n_s
        counts = torch.zeros(len(jobs), dtype=torch.int64, device="cuda")
        plan = hj.BatchPlan(jobs, counts)
        return {"case": c, "jobs": jobs, "counts": counts, "plan": plan, "ws": plan.workspace()}
    rk, rr, sk, sr = relations(c, seed)
    out_r, out_s = columns(room(c))
    st = {"case": c, "p": params_of(c), "rel": (rk, rr, sk, sr), "out": (out_r, out_s),
          "counts": torch.zeros(1, dtype=torch.int64, device="cuda")}
    if c["form"] == "join":
        st["ws"] = hj.workspace(st["p"], c["n_r"], c["n_s"])
        return st
    st["table_ws"] = torch.empty(hj.hj_table_bytes(st["p"], c["n_r"]), dtype=torch.uint8, device="cuda")
    st["table"] = hj.hj_build(st["p"], rk, rr, st["table_ws"])
    st["ws"] = torch.empty(hj.hj_probe_workspace_bytes(st["table"], c["n_s"]), dtype=torch.uint8, device="cuda")
    return st


def padded(joins, length):
    n = sum(j.numel() for j in joins)
    return torch.cat([*joins, torch.full((length - n,), -1, dtype=torch.int64, device="cuda")])


class Pairs(dict):
    """The result columns of one or more joins.  A join gives its pairs as a
    multiset in no fixed order, so reading them here sorts each join's pairs by
    (S row, R row); a program that goes on with the columns as they are sorts
    nothing.  "pairs": rid_s << 32 | rid_r of every join's pairs in turn, then
    -1 up to the columns' length; "counts": the pairs of each join."""

    def __init__(self, outs, counts):
        super().__init__(counts=counts, pairs=None)
        self.outs = outs

    def __getitem__(self, k):
        if k != "pairs":
            return super().__getitem__(k)
        got = []
        for (o_r, o_s), n in zip(self.outs, super().__getitem__("counts").tolist()):
            if not 0 <= n <= o_r.numel():
                raise ValueError("%d pairs in a result of %d" % (n, o_r.numel()))
            got.append(((o_s[:n].long() << 32) | o_r[:n].long()).sort().values)
        return padded(got, sum(o_r.numel() for o_r, _ in self.outs))


def run(st):
    form = st["case"]["form"]
    if form == "batch":
        st["plan"].run(st["ws"])
        return Pairs([j[4:6] for j in st["jobs"]], st["counts"])
    rk, rr, sk, sr = st["rel"]
    if form == "join":
        hj.hj_join(st["p"], rk, rr, sk, sr, *st["out"], st["ws"], st["counts"])
    else:
        if form == "build_probe":
            st["table"] = hj.hj_build(st["p"], rk, rr, st["table_ws"])
        hj.hj_probe(st["table"], sk, sr, *st["out"], st["ws"], st["counts"])
    return Pairs([st["out"]], st["counts"])


def work(c):
    """Every key and rid of R and S read once, every pair written once; a kept table's R is read too (its keys
    and the rids of the matches are needed by every probe)."""
    n = sum(s.n_r + s.n_s for s in job_specs(c, 0)) if c["form"] == "batch" else c["n_r"] + c["n_s"]
    return {"bytes": 8.0 * n + 8.0 * expected_pairs(c), "flops": 0.0}


def plain_join(rk, rr, sk, sr):
    """The sorted pairs by a sort of R and two binary searches per S tuple."""
    key, order = torch.sort(rk, stable=True)
    lo = torch.searchsorted(key, sk)
    n = torch.searchsorted(key, sk, right=True) - lo
    s = torch.repeat_interleave(torch.arange(sk.numel(), device=sk.device), n)
    first = torch.cumsum(n, 0) - n
    r = order[lo[s] + torch.arange(s.numel(), device=sk.device) - first[s]]
    return ((sr[s].long() << 32) | rr[r].long()).sort().values


def exact(c, seed):
    if c["form"] == "batch":
        rels = [(dgen.perm_keys(seed, s.r_stream, s.n_r), dgen.rows(s.n_r),
                 dgen.uniform_keys(seed, s.s_stream, s.n_s, s.s_domain), dgen.rows(s.n_s)) for s in job_specs(c, seed)]
        got = [plain_join(*r) for r in rels]
    else:
        got = [plain_join(*relations(c, seed))]
    return {"counts": torch.tensor([g.numel() for g in got], dtype=torch.int64), "pairs": padded(got, room(c))}
