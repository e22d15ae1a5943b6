"""The launch sequences of joins, builds and probes on the CPU: the built objects are linked
against recording HIP entry points (tests/host/launch_plan.cpp), nothing is launched."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_1307_1955_amd", "_build")
HIPCC = "/opt/rocm/bin/hipcc"
CLANGXX = "/opt/rocm/llvm/bin/clang++"
OBJECTS = ["engine.o", "costmodel.o", "scan.o", "shj.o", "phj_partition.o", "phj_join.o"]
SHJ, PHJ, AUTO = 0, 1, 2
ONE_PASS = 1


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    objs = [os.path.join(BUILD, o) for o in OBJECTS]
    if not (os.path.exists(HIPCC) and all(os.path.exists(o) for o in objs)):
        pytest.skip("hipcc or the library's objects are missing (run __graft_entry__.build() first)")
    d = tmp_path_factory.mktemp("launch_plan")
    drv, out = str(d / "driver.o"), str(d / "launch_plan")
    for cmd in ([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                 "-I", os.path.join(ROOT, "include"), "-c", os.path.join(ROOT, "tests", "host", "launch_plan.cpp"),
                 "-o", drv], [CLANGXX, "-o", out, drv, *objs]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
    return out


def launches(exe, mode, n_r, n_s, algo=PHJ, bits=(6, 6), tile=0, lds_cap=0, one_pass=False, env=None):
    """[(kernel, {field: value})] of the launches and the workspace bytes before them."""
    b = tuple(bits) + (0, 0)
    args = [mode, algo, len(bits), b[0], b[1], tile, lds_cap, ONE_PASS if one_pass else 0, n_r, n_s]
    r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, env={**os.environ, **(env or {})})
    assert r.returncode == 0 and "refused" not in r.stdout, r.stdout + r.stderr
    nbytes, seq = {}, []
    for ln in r.stdout.splitlines():
        w = ln.split()
        if "bytes" in w:
            nbytes[" ".join(w[:-2]) or mode] = int(w[-1])
        else:
            seq.append((w[0], dict((f.split("=") + [True])[:2] for f in w[1:])))
    return seq, nbytes


@pytest.mark.parametrize("bits", [(6, 6), (3,), (13,), (7, 6), (8, 8)])
@pytest.mark.parametrize("mode", ["join", "build", "probe"])
def test_injected_stall_spares_the_join_plan(exe, mode, bits):
    """The join plan's records are read without a clamp: its scan keeps the full poll bound and
    publishes its first tile, while the scans of the partition starts stall."""
    seq, _ = launches(exe, mode, 100000, 900000, bits=bits, env={"HJ_DEBUG_FAIL_PHASE": "scan_stall"})
    plans = [f["plan"] for _, f in seq if "plan" in f]
    assert plans and set(plans) == {"%d/0" % (1 << 20)}
    assert {f["scan"] for k, f in seq if k == "k_part_starts"} <= {"64/1"}


# (mode, |R|, |S|, options, bytes that were enough before two passes could be one scatter)
ENOUGH = [
    ("join", 1 << 20, 1 << 24, dict(algo=AUTO), 166010368),
    ("join", 390000, 22800000, dict(algo=AUTO), 196460544),
    ("join", 1 << 24, 1 << 24, dict(bits=(6, 6)), 891502336),
    ("join", 100000, 100000, dict(bits=(1, 2)), 5231872),
    ("join", 5000, 300, dict(bits=(9, 8)), 15485952),
    ("join", 48000, 700, dict(bits=(13,), tile=1024), 3838464),
    ("join", 5749, 281242, dict(bits=(5, 7), tile=1024), 6472960),
    ("build", 1200000, 1, dict(bits=(2, 10), tile=1024), 24702464),
    ("build", 66791, 1, dict(bits=(6, 6), tile=1024), 1899008),
    ("build", 42, 1, dict(bits=(13,), lds_cap=4096), 937728),
    ("build", 3400000, 1, dict(bits=(7, 6)), 62791168),
]


@pytest.mark.parametrize("case", range(len(ENOUGH)))
def test_workspaces_have_not_grown(exe, case):
    """A program's or a server slot's fixed workspace stays enough for the calls it was enough for."""
    mode, n_r, n_s, kw, enough = ENOUGH[case]
    assert launches(exe, mode, n_r, n_s, **kw)[1][mode] <= enough


@pytest.mark.parametrize("n_r,n_s", [(1 << 20, 15 << 20), (1 << 20, 1 << 24), (390000, 22800000), (1 << 21, 1 << 24),
                                     (1 << 22, 3 << 22), (1 << 23, 1 << 23)])
def test_auto_reserves_one_copy_for_one_scatter(exe, n_r, n_s):
    """HJ_AUTO's plans of up to 12 bits move the tuples once and reserve one copy (8 bytes a tuple,
    20 bytes a row of R for its tables, and the plan's small parts)."""
    seq, nbytes = launches(exe, "join", n_r, n_s, algo=AUTO)
    assert sum(k == "k_part_scatter" for k, _ in seq) == 1
    assert nbytes["join"] < 8 * (n_r + n_s) + 20 * n_r + (8 << 20)


@pytest.mark.parametrize("bits,lds_cap", [((4,), 0), ((8,), 256), ((6, 6), 256)])
def test_few_tuples_probing_a_large_table_clear_it_with_the_whole_device(exe, bits, lds_cap):
    """One tile of S: the scatter that clears the table's partitions has a workgroup per CU."""
    seq, _ = launches(exe, "probe", 1 << 24, 1000, bits=bits, lds_cap=lds_cap)
    scatters = [f for k, f in seq if k == "k_part_scatter"]
    assert len(scatters) == 1 and "clears" in scatters[0] and int(scatters[0]["grid"]) >= 256


# (|R|, bits, lds_cap, whether a launch before the join builds the HBM tables)
BUILDS = [(1 << 26, (6, 6), 0, True), (1 << 24, (6,), 0, True), (1 << 13, (5,), 256, True), (7500, (5,), 256, True),
          (1 << 25, (6, 6), 0, True), (1 << 24, (6, 6), 0, False), (1 << 20, (8,), 0, False), (6000, (5,), 256, False),
          (200, (1,), 256, False)]


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("case", range(len(BUILDS)))
def test_expected_tables_are_built_before_the_join(exe, case, one_pass):
    """Mean partitions near or past lds_cap: most have a table, built by a launch that fills the device;
    else the first join launch builds the few that a skewed R has."""
    n_r, bits, cap, before = BUILDS[case]
    for mode in ("join", "probe"):
        seq = [k for k, _ in launches(exe, mode, n_r, 100000, bits=bits, lds_cap=cap, one_pass=one_pass)[0]]
        assert ("k_ovf_build" in seq) == before
        assert not before or seq.index("k_ovf_build") + 1 == seq.index("k_join_write" if one_pass else "k_join_count")


def test_histogram_of_few_tuples_clears_with_more_workgroups(exe):
    """4096 rows into 2^18 partitions: one tile, and 2 MB of counts to clear."""
    seq, _ = launches(exe, "build", 4096, 1, bits=(9, 9))
    assert seq[0][0] == "k_part_hist" and int(seq[0][1]["grid"]) >= 64
    seq, _ = launches(exe, "join", 1 << 20, 1 << 20, bits=(6, 6))
    assert int(seq[0][1]["grid"]) == 512


# (tile, |R| + |S|, bits, tuples per scatter workgroup): requested tiles are the least, as include/hj.h has it
TILES = [(1024, (1 << 19) - 2, (6,), 1024), (1024, 1 << 19, (6,), 2048), (1024, 1 << 20, (6,), 4096), (2048, 1 << 22, (6,), 4096),
         (1024, 1 << 20, (6, 6), 4096), (4096, 1 << 22, (6,), 4096), (8192, 1 << 18, (6,), 8192), (4096, 1 << 21, (10,), 8192),
         (4096, (1 << 21) - 2, (10,), 4096)]


@pytest.mark.parametrize("case", range(len(TILES)))
def test_scatter_tiles(exe, case):
    tile, n, bits, want = TILES[case]
    seq, _ = launches(exe, "join", n // 2, n // 2, bits=bits, tile=tile)
    f = [f for k, f in seq if k == "k_part_scatter"][0]
    tiles = 2 * -(-(n // 2) // want)
    assert tiles <= int(f["grid"]) < tiles + 20  # (and the join plan's workgroups)


@pytest.mark.parametrize("n_r,n_s", [(8800, 15590469), (13212, 15941266), (300000, 4800000)])
def test_auto_keeps_one_table_for_a_small_lds_cap(exe, n_r, n_s):
    """Partitions that would all need HBM tables are not worth a partitioning of a small R."""
    for one_pass in (True, False):
        seq, _ = launches(exe, "join", n_r, n_s, algo=AUTO, lds_cap=256, one_pass=one_pass)
        assert "k_shj_build" in [k for k, _ in seq]
