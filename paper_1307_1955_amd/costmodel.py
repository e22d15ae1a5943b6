"""Per-step cost model of a join on MI355X (Section 4, Eq. 2-3), for planning.

The paper's abstract model sums, over the steps of a step series, each step's
computation time, memory-stall time and pipelined delay behind the previous
step, and takes the longer of the two processors.  Here one GPU runs every
step and a step is one kernel launch of the plan (the launch sequence of
csrc/engine.cpp), so

    T = sum over launches k of  D + d + max(M_k, W_k)

with D the delay of a dependent launch (its start behind the previous
kernel's end), d a kernel's fixed ramp-up and drain, M_k the launch's algorithmic bytes over the bandwidth its
access pattern reaches (streaming, scatter by run length, random table
lines), and W_k the latency term of its workgroups: ceil(workgroups / resident
slots) rounds of one workgroup's duration.  The computation term of Eq. 2 is
folded into W_k and into the per-tuple costs of the random-access steps; those
constants, like the bandwidths, are calibrated on the device (``tune.py
--collect`` records per-kernel HIP-event times over a grid of joins, ``fit``
fits each kernel's constants).  The same formulas are compiled into the
library (csrc/costmodel.cpp, constants from tuning/mi355x_calib.json via
tuning/calib_mi355x.inc), where HJ_AUTO evaluates them; a CPU test keeps the
two in agreement.
"""
from __future__ import annotations

import json
import math
import os

PKG = os.path.dirname(os.path.abspath(__file__))
CALIB_JSON = os.path.join(PKG, "tuning", "mi355x_calib.json")
CALIB_INC = os.path.join(PKG, "csrc", "calib_mi355x.inc")

CUS = 256
LDS_PER_CU = 160 * 1024
JOIN_CHUNK = 9216          # S tuples per join work item
OVF_CHUNK = 2048           # R tuples per HBM-table build item,
OVF_CHUNK_BIG = 16384      #   in a partition of more than OVF_BIG_PART tuples
OVF_BIG_PART = 1 << 16
OVF_GRID = 2048            # workgroups of the HBM-table clear launch
SHJ_TILE = 2048            # S tuples per SHJ probe workgroup
SCAN_CHUNK = 2048          # entries per scan workgroup
COUNTED_MAX_BITS = 13      # counted_pass2
WIDE_COUNT_BITS = 15       # the histogram counts the final partitions, from 400 tuples per partition on, up to here
FUSE_BITS = 12             # radix bits up to which one scatter makes the final partitions
SELF_BITS, SELF_WORDS = 8, 16384  # starts summed by the scatter's workgroups (csrc/hj_internal.h self_starts)

# the fitted constants, in this order (seconds, bytes/s; positive except SIGNED)
PARAMS = [
    "d_gap",               # delay of a dependent launch behind the previous kernel
    "d_kernel",            # fixed ramp-up and drain of a kernel
    "bw_hist", "t_hist_tile",
    "t_count_bin",         # a histogram workgroup: clear and write one counter
    "l_starts", "t_start_entry",  # the starts launch: its chain of waits, a count of a row summed
    "t_self_word",         # a scatter workgroup that sums the rows itself: a count of them
    "bw_scatter", "run_half", "t_scatter_tile",
    "t_reserve",           # a scatter tile: one partition's count, scan and reservation
    "p_part",              # the partitioning kernels overlap memory and latency imperfectly: (M^p + W^p)^(1/p)
    "q_part",              # share of a later round of partitioning tiles whose latency shows (rounds overlap)
    "t_scan_entry",
    "bw_join", "l_join0", "l_join_r", "l_join_s",
    "f_count", "f_1pass",  # a work item's latency in the count pass and the one-pass write, against the write pass
    "t_out",               # one reservation on the output count: they serialize (one per item and probe round)
    "p_join",              # the join kernels overlap memory and latency imperfectly: (M^p + W^p)^(1/p)
    "l_hbm0", "l_hbm_s", "t_ovf_insert", "l_ovf_round",
    "bw_fill",
    # random table accesses: throughput n * t * (table MiB)^gamma, at least a
    # latency floor t_round * (table / 32 KiB)^gamma_round (one round of
    # dependent accesses per resident lane, slower as fewer lines hit the caches)
    "t_ins", "gamma_ins", "t_bround", "gamma_bround",
    "t_probe", "gamma_probe", "t_pround", "gamma_pround", "t_match",
]
# may be negative: back-to-back launches overlap (d_gap); the per-access cost
# may fall with the table size while the chip fills (the exponents)
SIGNED = {"d_gap", "gamma_ins", "gamma_bround", "gamma_probe", "gamma_pround"}


def load(path: str = CALIB_JSON) -> dict:
    with open(path) as f:
        return json.load(f)["params"]


SHJ_SLOTS_PER_ROW = 2.0  # csrc/hj_internal.h kShjSlotsPerRow


def shj_slots(n_r: int) -> int:
    s = int(SHJ_SLOTS_PER_ROW * max(n_r, 1) + 0.999999)
    return (s + 15) // 16 * 16


def scatter_tile(tile: int, bits: int, n: int) -> int:
    """Tuples per scatter workgroup (csrc/hj_internal.h scatter_tile)."""
    while tile < 4096 and n >= 512 * tile:
        tile *= 2
    want = 16384 if bits == 12 else 8192 if bits >= 10 else tile
    return tile if tile < 4096 or want <= tile or n < 256 * want else want


def _part_block(tile: int) -> int:
    return 1024 if tile >= 8192 else 512 if tile >= 4096 else 256


def _scatter_slots(bits: int, tile: int) -> int:
    P = 1 << bits
    lds = 8 * (tile + 64) + 4 * (max(P, 64) + 128)
    by_lds = LDS_PER_CU // lds
    by_threads = 2048 // _part_block(tile)
    return CUS * max(1, min(by_lds, by_threads))


def hist_grid(tiles: int, count_bits: int) -> int:
    """Workgroups of the histogram (csrc/hj_internal.h hist_rows)."""
    cap = 256 if count_bits > 13 else 512 if count_bits > 10 else 1024
    g = 8 if tiles >= 64 else 1
    while 2 * g <= cap and 2 * g <= tiles:
        g *= 2
    return g


def join_lds_bytes(cap: int) -> int:
    heads = 64
    while 2 * heads <= cap:
        heads *= 2
    if 4 * (2 * heads + 2 * (cap + 128)) <= LDS_PER_CU // 3 - 1536:
        heads *= 2
    return 4 * (heads + 2 * (cap + 128))


def join_slots(cap: int) -> int:
    """Join work items resident at once: workgroups per CU by LDS and by the
    waves the kernels' register budget allows (6 per SIMD, 4 with the largest
    build), 512-thread workgroups."""
    by_waves = (4 if cap > 4608 else 6) * 4 // 8
    return CUS * max(1, min(LDS_PER_CU // (join_lds_bytes(cap) + 512), by_waves))


def direct_blocks(cap: int) -> int:
    """Workgroups of a direct join that a CU holds, without rids in LDS where that
    holds more (csrc/phj_join.hip direct_blocks)."""
    heads = 64
    while 2 * heads <= cap:
        heads *= 2
    by_lds = LDS_PER_CU // (4 * (2 * heads + cap + 128) + 512)
    return max(1, min(by_lds, (4 if cap > 4608 else 6) * 4 // 8))


def _nonempty(mean: float) -> float:
    return 1.0 - math.exp(-mean) if mean < 30 else 1.0


def _smooth_max(a: float, b: float, p: float) -> float:
    """(a^p + b^p)^(1/p): max(a, b) as p grows, more than it when a and b are close."""
    m = max(a, b)
    if m <= 0.0:
        return 0.0
    return m * ((a / m) ** p + (b / m) ** p) ** (1.0 / p)


def _table_factor(table_bytes: float, gamma: float, base: float = 1 << 20) -> float:
    """Change of a random access's cost with the table size (1 up to base bytes)."""
    return (max(table_bytes, base) / base) ** gamma


def counted_pass2(passes: int, b1: int, b2: int) -> bool:
    """Two passes of 4..13 bits in all (csrc/hj_internal.h)."""
    return passes == 2 and 4 <= b1 + b2 <= COUNTED_MAX_BITS


def one_scatter(passes: int, b1: int, b2: int) -> bool:
    return passes == 1 or b1 + b2 <= FUSE_BITS


def counts_final(passes: int, b1: int, b2: int, n: int) -> bool:
    """Whether the first histogram counts the final partitions."""
    return one_scatter(passes, b1, b2) or (b1 + b2 <= WIDE_COUNT_BITS and n >= 400 << (b1 + b2))


def tables_expected(n_r: int, P: int, cap: int) -> bool:
    """Whether a launch of its own builds the HBM tables (csrc/hj_internal.h)."""
    mean = n_r / P
    return n_r > cap and mean + 3.0 * math.sqrt(mean) > cap


def ovf_chunk(r_part: float) -> int:
    c = OVF_CHUNK
    if r_part > OVF_BIG_PART:
        while c < OVF_CHUNK_BIG and c < math.floor(r_part / 128):
            c *= 2
    return c


def launches(plan: dict, n_r: int, n_s: int, m: float) -> list[tuple[str, dict]]:
    """The launch sequence of a join (engine.cpp) with each launch's features.
    plan: resolved parameters: algo ("shj"/"phj"), passes, bits (b1, b2), tile,
    lds_cap, one_pass."""
    n = n_r + n_s
    out = []
    if n_r == 0 or n_s == 0:
        return [("zero_count", {})]
    if plan["algo"] == "shj":
        slots = shj_slots(n_r)
        tb = 8.0 * slots
        out.append(("shj_fill", {"bytes": 8.0 * slots}))
        out.append(("shj_build", {"n": n_r, "tb": tb}))
        if plan["one_pass"]:
            out.append(("shj_write_1pass", {"n": n_s, "tb": tb, "m": m}))
        else:
            tiles = math.ceil(n_s / SHJ_TILE)
            out.append(("shj_count", {"n": n_s, "tb": tb}))
            out.append(("scan_u64", {"entries": 4 * tiles}))
            out.append(("shj_write", {"n": n_s, "tb": tb, "m": m}))
        return out
    cap = plan["lds_cap"]
    if plan["passes"] == 0:
        slots = CUS * direct_blocks(cap)
        chunk = JOIN_CHUNK // 2 if n_s <= slots * (JOIN_CHUNK // 2) else JOIN_CHUNK
        items = math.ceil(n_s / chunk)
        if items > 1:
            out.append(("zero_count", {}))
        out.append(("direct_join", {"items": items, "grid": items, "r": n_r, "s": min(n_s, chunk), "cap": cap,
                                    "bytes": 8.0 * n + 8.0 * m, "hbm": 0}))
        return out
    tile = plan["tile"]
    b1, b2 = plan["bits"][0], (plan["bits"][1] if plan["passes"] == 2 else 0)
    B = b1 + b2
    P = 1 << B
    P1 = 1 << b1
    one = one_scatter(plan["passes"], b1, b2)
    final = counts_final(plan["passes"], b1, b2, n)
    tile1 = scatter_tile(tile, B if one else b1, n)
    tiles1 = math.ceil(n_r / tile1) + math.ceil(n_s / tile1)
    self_starts = one and B <= SELF_BITS and (tiles1 << B) <= min(SELF_WORDS, 32 * _part_block(tile1))
    cbits = B if final else b1  # what the histogram counts
    grid = tiles1 if self_starts else hist_grid(tiles1, cbits)
    out.append(("part_hist", {"n": n, "grid": grid, "bins": 1 << cbits}))
    if not self_starts:
        out.append(("part_starts", {"entries": 2.0 * grid * ((1 << cbits) + (P1 if final and not one else 0))}))
    r_part, s_part = n_r / P, n_s / P
    hbm = r_part > cap
    ovf_r = n_r if hbm else 0
    clears = one or (final and b2 <= 6)  # the last scatter clears the HBM tables
    cleared = 16.0 * ovf_r if clears else 0.0
    out.append(("part_scatter", {"n": n, "tiles": tiles1, "tile": tile1, "bits": B if one else b1,
                                 "extra": cleared if one else 0.0,
                                 "words": float(tiles1 << B) if self_starts else 0.0}))
    if not one:
        tile2 = scatter_tile(tile, b2, n)
        seg = n / (2.0 * P1)
        tiles2 = 2 * P1 * max(1, math.ceil(seg / tile2)) if seg > 0 else 0
        if not final:
            out.append(("part_hist2", {"n": 2.0 * n, "grid": tiles2, "bins": 1 << b2}))
            out.append(("scan_u32", {"entries": 2.0 * P}))
        out.append(("part_scatter", {"n": n, "tiles": tiles2, "tile": tile2, "bits": b2, "extra": cleared,
                                     "words": 0.0}))
    pairs = P * _nonempty(r_part) * _nonempty(s_part)
    items = pairs * max(1, math.ceil(s_part / JOIN_CHUNK))
    grid = P + math.ceil(n_s / JOIN_CHUNK)
    s_item = min(max(s_part, 1.0), JOIN_CHUNK)
    chunk = ovf_chunk(r_part)
    # HBM tables are built by the first join launch, or one before it
    build = {"ovf_n": ovf_r, "ovf_items": P * math.ceil(r_part / chunk) if hbm else 0, "per": min(r_part, chunk)}
    if not clears:
        out.append(("ovf_clear", {"bytes": 16.0 * ovf_r}))
    if tables_expected(n_r, P, cap):
        out.append(("ovf_build", build))
        build = {}
    jf = {"items": items, "grid": grid, "r": min(r_part, cap), "s": s_item, "cap": cap, "hbm": int(hbm)}
    if not plan["one_pass"]:
        out.append(("join_count", dict(jf, bytes=4.0 * n, **build)))
        out.append(("scan_u64", {"entries": 8 * grid}))
        out.append(("join_write", dict(jf, bytes=8.0 * n + 8.0 * m)))
    else:
        out.append(("join_write_1pass", dict(jf, bytes=8.0 * n + 8.0 * m, **build)))
    return out


def _part_lat(rounds: int, per_tile: float, c: dict) -> float:
    """Latency term of a partitioning launch: the first round of tiles, then a
    share q_part of each later round (rounds overlap)."""
    return per_tile * (1.0 + (rounds - 1) * c["q_part"])


def _build_seconds(f: dict, c: dict) -> float:
    """Building the HBM tables: inserts, or rounds of items of ovf_chunk() tuples."""
    if not f.get("ovf_items"):
        return 0.0
    turns = math.ceil(f["ovf_items"] / (3.0 * CUS))
    return max(f["ovf_n"] * c["t_ovf_insert"], turns * math.ceil(f["per"] / 512.0) * c["l_ovf_round"])


def kernel_seconds(name: str, f: dict, c: dict) -> float:
    """One kernel's duration: ramp-up/drain + max(memory term, workgroup-latency term)."""
    d = c["d_kernel"]
    if name in ("part_hist", "part_hist2"):
        if f["grid"] == 0:
            return d
        per = c["t_hist_tile"] * (f["n"] / f["grid"]) / 8192.0 + c["t_count_bin"] * f["bins"]
        return d + _smooth_max(4.0 * f["n"] / c["bw_hist"], _part_lat(math.ceil(f["grid"] / 1024.0), per, c),
                               c["p_part"])
    if name == "part_starts":
        return d + c["l_starts"] + f["entries"] * c["t_start_entry"]
    if name == "part_scatter":
        if f["tiles"] == 0:
            return d
        run = f["tile"] / float(1 << f["bits"])
        bw = c["bw_scatter"] * run / (run + c["run_half"])
        rounds = math.ceil(f["tiles"] / _scatter_slots(f["bits"], f["tile"]))
        per_tile = (c["t_scatter_tile"] * f["tile"] / 8192.0 + c["t_reserve"] * (1 << f["bits"]) / 4096.0 +
                    c["t_self_word"] * f["words"])
        return d + _smooth_max((16.0 * f["n"] + f["extra"]) / bw, _part_lat(rounds, per_tile, c), c["p_part"])
    if name in ("scan_u32", "scan_u64"):
        return d + f["entries"] * c["t_scan_entry"]
    if name in ("join_count", "join_write", "join_write_1pass", "direct_join"):
        if f["hbm"]:
            lat = c["l_hbm0"] + c["l_hbm_s"] * f["s"]
        else:
            lat = c["l_join0"] + c["l_join_r"] * f["r"] + c["l_join_s"] * f["s"]
        lat *= c["f_count"] if name == "join_count" else c["f_1pass"] if name == "join_write_1pass" else 1.0
        rounds = math.ceil(max(f["items"], 1) / join_slots(f["cap"]))
        build = _build_seconds(f, c)
        # the first round, then its later ones beside the memory traffic
        t = lat + _smooth_max(f["bytes"] / c["bw_join"], (rounds - 1) * lat, c["p_join"])
        if name == "join_write_1pass":
            t = _smooth_max(t, f["items"] * math.ceil(f["s"] / (JOIN_CHUNK / 2)) * c["t_out"], 4.0)
        return d + build + t
    if name == "ovf_build":
        return d + _build_seconds(f, c)
    if name == "ovf_clear":
        return d + f["bytes"] / c["bw_fill"]
    if name == "shj_fill":
        return d + f["bytes"] / c["bw_fill"]
    if name == "shj_build":
        floor = c["t_bround"] * _table_factor(f["tb"], c["gamma_bround"], 32768.0)
        return d + max(f["n"] * c["t_ins"] * _table_factor(f["tb"], c["gamma_ins"]), floor)
    if name in ("shj_count", "shj_write", "shj_write_1pass"):
        t = f["n"] * c["t_probe"] * _table_factor(f["tb"], c["gamma_probe"])
        if name != "shj_count":
            t += f["m"] * c["t_match"]
        return d + max(t, c["t_pround"] * _table_factor(f["tb"], c["gamma_pround"], 32768.0))
    return d  # small set-up kernels: the delay alone


def join_seconds(plan: dict, n_r: int, n_s: int, m: float, c: dict) -> float:
    ls = launches(plan, n_r, n_s, m)
    return sum(kernel_seconds(k, f, c) for k, f in ls) + len(ls) * c["d_gap"]


# starting point of the fit: rough MI355X figures
START = {
    "d_gap": 2e-6, "d_kernel": 3e-6, "bw_hist": 4.5e12, "t_hist_tile": 5e-6, "t_count_bin": 1e-9, "l_starts": 4e-6, "t_start_entry": 1e-12, "t_self_word": 1e-10,
    "bw_scatter": 5.2e12, "run_half": 8.0, "t_scatter_tile": 12e-6, "t_reserve": 2e-6, "p_part": 4.0, "q_part": 0.5, "t_scan_entry": 2e-12, "bw_join": 4e12, "l_join0": 4e-6, "l_join_r": 1e-9,
    "l_join_s": 5e-10, "f_count": 0.8, "f_1pass": 1.2, "t_out": 1e-8,  "p_join": 4.0, "l_hbm0": 8e-6, "l_hbm_s": 2e-9, "t_ovf_insert": 1e-10, "l_ovf_round": 4e-6,
    "bw_fill": 5e12, "t_ins": 1e-10, "gamma_ins": -0.2, "t_bround": 1e-5, "gamma_bround": 0.1,
    "t_probe": 3e-11, "gamma_probe": 0.0, "t_pround": 2e-5, "gamma_pround": 0.1, "t_match": 1e-11,
}


def fit(raw: dict) -> tuple[dict, dict]:
    """Fits the constants to per-kernel HIP-event times (``tune.py --collect``
    records): least squares on log(predicted / measured) over every launch, then
    the launch gap from the whole-join times.  Returns (params, fit report)."""
    import numpy as np
    from scipy.optimize import least_squares

    pts = []  # (kernel name, features, measured seconds)
    joins = []  # (launch list, measured kernel seconds list, whole join seconds)
    for r in raw["records"]:
        rs = r["resolved"]
        plan = {"algo": "shj" if rs["algo"] == 0 else "phj", "passes": rs["passes"], "bits": tuple(rs["bits"]),
                "tile": rs["tile"], "lds_cap": rs["lds_cap"], "one_pass": rs["one_pass"]}
        ls = launches(plan, r["cfg"]["n_r"], r["cfg"]["n_s"], r["pairs"])
        names = [k for k, _ in r["kernels"]]
        if names != [k for k, _ in ls]:
            raise ValueError("launch sequence of %r: recorded %s, modelled %s" % (r["cfg"], names, [k for k, _ in ls]))
        for (k, f), (_, ms) in zip(ls, r["kernels"]):
            pts.append((k, f, max(ms, 1e-4) * 1e-3))
        joins.append((plan, r["cfg"]["n_r"], r["cfg"]["n_s"], r["pairs"], r["join_ms"] * 1e-3, len(ls)))
    free = [k for k in PARAMS if k != "d_gap"]
    signed = [k in SIGNED for k in free]

    def params_of(x):
        c = {k: float(v if sg else np.exp(v)) for k, v, sg in zip(free, x, signed)}
        c["d_gap"] = 0.0
        return c

    def x_of(c):
        return np.array([c[k] if sg else math.log(c[k]) for k, sg in zip(free, signed)])

    def resid(x):
        c = params_of(x)
        return np.array([math.log(kernel_seconds(k, f, c) / t) for k, f, t in pts])

    sol = least_squares(resid, x_of(START), method="trf", max_nfev=4000)
    c = params_of(sol.x)
    # the launch gap: what whole joins take beyond their kernels' event times
    gaps = [(t - sum(kernel_seconds(k, f, c) for k, f in launches(plan, nr, ns, m))) / nl
            for plan, nr, ns, m, t, nl in joins]
    c["d_gap"] = float(np.median(gaps))
    r = resid(sol.x)
    err = [join_seconds(plan, nr, ns, m, c) / t - 1.0 for plan, nr, ns, m, t, nl in joins]
    report = {"launches": len(pts), "joins": len(joins),
              "kernel_abs_log_err_median": float(np.median(np.abs(r))),
              "kernel_abs_log_err_p90": float(np.percentile(np.abs(r), 90)),
              "join_abs_rel_err_median": float(np.median(np.abs(err))),
              "join_abs_rel_err_p90": float(np.percentile(np.abs(err), 90)),
              "join_within_15pct": float(np.mean(np.abs(err) <= 0.15))}
    return {k: c[k] for k in PARAMS}, report


def plan_of(resolved) -> dict:
    """Plan dict from a resolved HjParams (hj_resolve_params)."""
    return {"algo": "shj" if resolved.algo == 0 else "phj", "passes": int(resolved.passes),
            "bits": (int(resolved.bits[0]), int(resolved.bits[1])), "tile": int(resolved.tile),
            "lds_cap": int(resolved.lds_cap), "one_pass": bool(resolved.flags & 1)}


def write_inc(params: dict, path: str = CALIB_INC) -> None:
    """The constants as a C++ include for csrc/costmodel.cpp (generated; do not edit)."""
    lines = ["// Generated by paper_1307_1955_amd.costmodel.write_inc from tuning/mi355x_calib.json;",
             "// the per-step cost model's constants calibrated on MI355X.  Do not edit."]
    for k in PARAMS:
        lines.append("constexpr double k_%s = %.17g;" % (k, params[k]))
    with open(path, "w") as f:
        f.write("\n".join(lines) + "\n")
