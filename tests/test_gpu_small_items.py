"""GPU parity of join items on both sides of the small-item rule (up to 512 R and 1024 S tuples
of a partition): one partition of either kind beside the other, few and many link bits."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1307_1955_amd.hj as hj  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("lds_cap", [1024, 8192])
@pytest.mark.parametrize("r_len", [(512, 513), (1, 511), (64, 65)])
@pytest.mark.parametrize("s_len", [(1024, 1025), (1, 1023), (512, 513), (64, 4608), (9216, 65)])
@pytest.mark.parametrize("dup", [1, 40])
def test_small_items(dup, s_len, r_len, lds_cap, one_pass):
    rng = np.random.default_rng(r_len[0] * 10007 + s_len[0] * 13 + dup)
    # partition p (the key's low bit) holds r_len[p] R rows and s_len[p] S rows
    dom = [max(1, n // dup) for n in r_len]
    rk = np.concatenate([2 * rng.integers(0, dom[p], r_len[p]) - 2 ** 31 + p for p in (0, 1)])
    sk = np.concatenate([2 * rng.integers(0, dom[p] + 3, s_len[p]) - 2 ** 31 + p for p in (0, 1)])
    rk, sk = (a[rng.permutation(len(a))].astype(np.int32) for a in (rk, sk))
    rr = rng.permutation(len(rk)).astype(np.int32) * 3 - 7
    sr = rng.permutation(len(sk)).astype(np.int32) + 11
    want = oracle.canonical(*oracle.join(rk, rr, sk, sr))
    t = [torch.from_numpy(a).to(DEV) for a in (rk, rr, sk, sr)]
    o_r, o_s, cnt = hj.join(*t, p=hj.params("phj", 1, (1,), lds_cap=lds_cap, one_pass=one_pass), capacity=len(want))
    assert cnt == len(want)
    assert np.array_equal(oracle.canonical(o_r.cpu().numpy(), o_s.cpu().numpy()), want)
