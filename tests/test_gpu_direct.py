"""GPU parity of single direct joins (R fits one LDS table) where their launches change:
one work item, which clears the count and the error word itself, and more; S chunks of one
probe round and of two (csrc/hj_internal.h direct_chunk).  Integer results: exact equality."""
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
ROUND = 4608


@pytest.mark.parametrize("n_r,n_s", [(1, 1), (300, ROUND), (300, ROUND + 1), (2049, 2 * ROUND + 1),
                                     (4608, 640 * ROUND), (4608, 640 * ROUND + 1), (8192, 256 * ROUND),
                                     (8192, 256 * ROUND + 1)])
def test_direct_chunks(n_r, n_s):
    r, s = gen.unique_uniform(7, n_r, n_s, 2 * n_r)
    t = [torch.from_numpy(a).to(DEV) for a in (r.key, r.rid, s.key, s.rid)]
    want = oracle.canonical(*oracle.join(r.key, r.rid, s.key, s.rid))
    p = hj.params("phj", 0)
    ws = hj.workspace(p, n_r, n_s)
    ws.fill_(0xFF)
    out = [torch.full((n_s,), -1, dtype=torch.int32, device=DEV) for _ in range(2)]
    count = torch.full((1,), 12345, dtype=torch.int64, device=DEV)
    for _ in range(2):  # (the second call finds the first one's count)
        hj.hj_join(p, *t, *out, ws, count)
        assert int(count) == len(want)
        assert np.array_equal(oracle.canonical(*[o[: len(want)].cpu().numpy() for o in out]), want)
