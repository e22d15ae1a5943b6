"""GPU parity of direct joins with R's rids in LDS and in R's column: capacities on both sides of
the rule, few items (LDS) and more than the device holds at once."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1307_1955_amd.hj as hj  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n_s", [5000, 2_400_001, 4_800_000])
@pytest.mark.parametrize("n_r,dup", [(4032, 1), (4033, 1), (4096, 3), (4608, 1), (4609, 1), (5952, 2), (5953, 2), (8128, 1), (8129, 1),
                                     (8192, 5)])
def test_direct_rids(n_r, dup, n_s):
    rng = np.random.default_rng(n_r + n_s)
    rk = (rng.permutation(n_r) // dup - 5).astype(np.int32)
    sk = rng.integers(-10, 3 * n_r // dup, n_s).astype(np.int32)
    rr = (rng.permutation(n_r) * 2 - 9).astype(np.int32)
    sr = rng.permutation(n_s).astype(np.int32)
    t = [torch.from_numpy(a).to(DEV) for a in (rk, rr, sk, sr)]
    want = oracle.canonical(*oracle.join(rk, rr, sk, sr))
    o_r, o_s, cnt = hj.join(*t, p=hj.params("phj", 0, (0, 0)), capacity=len(want))
    assert cnt == len(want)
    assert np.array_equal(oracle.canonical(o_r.cpu().numpy(), o_s.cpu().numpy()), want)
