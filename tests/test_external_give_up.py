"""hj_join_external on the CPU after its partition pass gave up (tests/host/external_give_up.cpp):
boundaries that run backwards are not linked, and the call reports a device error."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_1307_1955_amd", "_build")
HIPCC = "/opt/rocm/bin/hipcc"
CLANGXX = "/opt/rocm/llvm/bin/clang++"
OBJECTS = ["external.o", "engine.o", "costmodel.o", "scan.o", "shj.o", "phj_partition.o", "phj_join.o"]
HJ_ERR_DEVICE = 4


def test_boundaries_of_a_pass_that_gave_up_are_not_linked(tmp_path):
    objs = [os.path.join(BUILD, o) for o in OBJECTS]
    if not (os.path.exists(HIPCC) and all(os.path.exists(o) for o in objs)):
        pytest.skip("hipcc or the library's objects are missing (run __graft_entry__.build() first)")
    drv, out = str(tmp_path / "driver.o"), str(tmp_path / "external_give_up")
    for cmd in ([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                 "-I", os.path.join(ROOT, "include"), "-c", os.path.join(ROOT, "tests", "host", "external_give_up.cpp"),
                 "-o", drv], [CLANGXX, "-o", out, drv, *objs, "-lm"]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    last = r.stdout.splitlines()[-1].split()
    assert "copy" not in r.stdout, r.stdout
    assert int(last[1]) == HJ_ERR_DEVICE and int(last[3]) >= 6 and int(last[5]) == 0, r.stdout
