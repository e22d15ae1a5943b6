"""A call whose chained scan gave up (HJ_DEBUG_FAIL_PHASE=scan_stall) neither builds nor looks
up the HBM tables of oversized partitions.  Only the scan of the match counts gives up here:
four partitions have one workgroup of starts, so the tables themselves are whole."""
import os

import numpy as np
import pytest

import oracle
from paper_1307_1955_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1307_1955_amd.hj as hj  # noqa: E402


@pytest.mark.parametrize("bits", [(2,), (1, 1)])
def test_no_table_is_walked_after_a_give_up(bits, monkeypatch):
    n_r, n_s = 20000, 3 << 20  # every partition of R is larger than 256; two tiles of counts to scan
    r, s = gen.unique_uniform(31, n_r, n_s, 2 * n_r)
    t = [torch.from_numpy(a).cuda() for a in (r.key, r.rid, s.key, s.rid)]
    p = hj.params("phj", len(bits), bits, lds_cap=256)
    ws = hj.workspace(p, n_r, n_s)
    out = [torch.full((n_s,), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
    d = torch.zeros(1, dtype=torch.int64, device="cuda")
    with monkeypatch.context() as m:
        m.setenv("HJ_DEBUG_FAIL_PHASE", "scan_stall")
        hj.hj_join(p, *t, *out, ws, d)
        with pytest.raises(hj.HJError):
            hj.hj_workspace_status(ws)
    assert "HJ_DEBUG_FAIL_PHASE" not in os.environ
    assert all(bool((o == -7).all()) for o in out)  # the write pass came after the give-up
    cnt = hj.hj_join_sync(p, *t, *out, ws, d)
    want = oracle.canonical(*oracle.join(r.key, r.rid, s.key, s.rid))
    assert cnt == len(want)
    assert np.array_equal(oracle.canonical(out[0][:cnt].cpu().numpy(), out[1][:cnt].cpu().numpy()), want)
