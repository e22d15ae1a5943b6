"""GPU parity of the histograms that count the final partitions of two scatters: the sums of a pass-1
partition's counters by a thread (fewer than 64 of them) or by a wave; and tiles raised to 4096."""
import numpy as np
import pytest

import oracle
from paper_1307_1955_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1307_1955_amd.hj as hj  # noqa: E402

DEV = torch.device("cuda:0")
CASES = [(1 << 20, 2500000, (1, 12)), (1 << 20, 2500000, (7, 6)), (1 << 20, 2500000, (8, 5)), (1 << 21, 5 << 20, (2, 12)),
         # too few tuples: a second histogram
         (1, 1, (7, 6)), (5000, 300, (7, 6)), (70001, 60001, (1, 12)), (70001, 60001, (12, 1)), (64 * 1024, 64 * 1024 - 1, (6, 7)),
         # twice the requested tile of 1024 from 2^19 tuples on, 4096 from 2^20, and one scatter of them
         (1 << 18, (1 << 18) - 1, (3, 4)), (1 << 18, 1 << 18, (3, 4)), (1 << 19, 1 << 19, (3, 4)), (1 << 19, (1 << 19) - 1, (6, 6))]


@pytest.mark.parametrize("tile", [0, 1024])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_wide_counts(case, tile):
    n_r, n_s, bits = CASES[case]
    r, s = gen.unique_uniform(20 + case, n_r, n_s, 2 * n_r)
    rk = r.key.copy()
    rk[: n_r // 8] = rk[n_r // 8: n_r // 8 * 2]
    t = [torch.from_numpy(a).to(DEV) for a in (rk, r.rid, s.key, s.rid)]
    p = hj.params("phj", 2, bits, one_pass=bool(case % 2), tile=tile)
    o_r, o_s, cnt = hj.join(*t, p=p, capacity=2 * n_s)
    want = oracle.canonical(*oracle.join(rk, r.rid, s.key, s.rid))
    assert cnt == len(want)
    assert np.array_equal(oracle.canonical(o_r.cpu().numpy(), o_s.cpu().numpy()), want)
