"""Chain lengths the LDS-table probe walks, and what grouping probes by key-list
length could save (Section 3.3, "workload divergence").

The join kernel builds, per work item, a chained table over R_i in LDS: 2^h
chain heads, h = floor(log2(lds_cap)) (4416 rows here), a record per R tuple
pushed on the chain of its bucket (the top h bits of the mixed radix hash
above the partition's bits); a probe walks the whole
chain of its S key's bucket.  A wave probes 9 S keys per lane in lockstep, so
a wave's round takes as many steps as the longest chain among its 576 keys.
The paper groups tuples of similar key-list length so that a wave's lanes
finish together.  This computes, exactly (same hash, same layout), the walk
length of every S tuple of a 2-pass 6+6-bit PHJ (identity radix hash) over the
16M x 16M workload and over the 16M x 64M Zipf workloads, the steps of every
wave round as the kernel forms them, and the steps the same waves would take
if each work item's S keys were first sorted by walk length (the best grouping
can do).

``python -m paper_1307_1955_amd.chains`` prints one JSON row per workload.
"""
from __future__ import annotations

import numpy as np

from . import gen

KSU = 9              # S keys per lane of a probe round
WAVE = 64
WAVES = 8
ROUND = KSU * WAVE * WAVES   # 4608 S keys per round of a work item
CHUNK = 2 * ROUND            # S keys per work item


def mixed(k: np.ndarray, bits: int) -> np.ndarray:
    """The LDS table's 32-bit mix of the key's radix hash (identity) above the
    partition's bits (csrc/phj_join.hip mixed())."""
    m, keep = np.uint64(0xFFFFFFFF), np.uint64((0xFFFFFFFF << bits) & 0xFFFFFFFF)
    h = ((k.astype(np.uint32).astype(np.uint64) & keep) * np.uint64(0x9E3779B1)) & m
    h ^= (h >> np.uint64(15)) & keep
    return (h * np.uint64(0x85EBCA6B)) & m


def walk_lengths(r_key: np.ndarray, s_key: np.ndarray, bits: int = 12, log2_heads: int = 12):
    """Per S tuple: its partition and the length of the chain its probe walks."""
    mask = np.int64((1 << bits) - 1)
    sp = s_key.astype(np.int64) & mask
    # global bucket id = partition * 2^log2_heads + bucket
    sh = np.uint64(32 - log2_heads)
    rb = (mixed(r_key, bits) >> sh).astype(np.int64)
    sb = (mixed(s_key, bits) >> sh).astype(np.int64)
    chain = np.bincount(((r_key.astype(np.int64) & mask) << log2_heads) + rb, minlength=1 << (bits + log2_heads))
    return sp, chain[(sp << log2_heads) + sb]


def wave_steps(sp: np.ndarray, walk: np.ndarray, grouped: bool) -> tuple[int, int]:
    """Total lockstep steps over all wave rounds, and the walked records, when
    S is partitioned (stable order inside a partition) and each work item's S
    keys go to the waves as the kernel assigns them (grouped: sorted by walk
    length first)."""
    order = np.argsort(sp, kind="stable")
    sp, walk = sp[order], walk[order]
    starts = np.searchsorted(sp, np.arange(sp.max() + 2))
    total = 0
    for i in range(len(starts) - 1):
        w = walk[starts[i]: starts[i + 1]]
        for c0 in range(0, len(w), CHUNK):
            item = w[c0: c0 + CHUNK]
            for r0 in range(0, len(item), ROUND):
                rnd = item[r0: r0 + ROUND]
                if grouped:
                    rnd = np.sort(rnd)
                # wave v of the round takes keys [v * 576, (v + 1) * 576)
                for v in range(0, len(rnd), KSU * WAVE):
                    total += int(rnd[v: v + KSU * WAVE].max())
    return total, int(walk.sum())


def report(n: int = 1 << 24) -> list[dict]:
    rows = []
    r, s = gen.config_c2(n=n)
    cases = [("C2 16M x 16M (uniform S over 1..2^25)", r.key, s.key)]
    for theta in (0.5, 1.0):
        r3, s3 = gen.config_c3(theta=theta, n_r=n, n_s=4 * n)
        cases.append(("C3 16M x 64M, Zipf theta %.1f" % theta, r3.key, s3.key))
    for name, rk, sk in cases:
        sp, walk = walk_lengths(rk, sk)
        hist = np.bincount(walk, minlength=8)
        steps, work = wave_steps(sp, walk, grouped=False)
        steps_g, _ = wave_steps(sp, walk, grouped=True)
        rows.append({"workload": name, "mean_walk": float(walk.mean()),
                     "walk_share": {str(k): float(hist[k] / len(walk)) for k in range(min(len(hist), 8))},
                     "max_walk": int(walk.max()), "lane_utilisation": work / (steps * KSU * WAVE),
                     "steps": steps, "steps_grouped": steps_g, "grouping_saves": 1 - steps_g / steps})
    return rows


if __name__ == "__main__":
    import json
    for row in report():
        print(json.dumps(row))
