"""GPU parity of builds with more hot keys than are recorded, and of heavy S tuples whose rows end
inside and on a scan step of 4096: SHJ and HBM-table partitions, both output modes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1307_1955_amd.hj as hj  # noqa: E402

DEV = torch.device("cuda:0")
PLANS = [dict(algo="shj"), dict(algo="phj", passes=1, bits=(1,), lds_cap=256), dict(algo="phj", passes=2, bits=(2, 3), lds_cap=256)]


def check(rk, sk, kw, one_pass, seed):
    rng = np.random.default_rng(seed)
    rr = rng.permutation(len(rk)).astype(np.int32)
    sr = rng.permutation(len(sk)).astype(np.int32)
    want = oracle.canonical(*oracle.join(rk, rr, sk, sr))
    t = [torch.from_numpy(a).to(DEV) for a in (rk, rr, sk, sr)]
    o_r, o_s, cnt = hj.join(*t, p=hj.params(one_pass=one_pass, **kw), capacity=len(want))
    assert cnt == len(want)
    assert np.array_equal(oracle.canonical(o_r.cpu().numpy(), o_s.cpu().numpy()), want)


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("plan", range(len(PLANS)))
@pytest.mark.parametrize("keys,rows", [(62, 300), (63, 300), (64, 300), (200, 90), (3, 5000)])
def test_hot_keys(keys, rows, plan, one_pass):
    """Runs of hot keys beside a few rows of others; keys are -1, 0 and their neighbours too."""
    rng = np.random.default_rng(keys * 31 + rows)
    rk = np.concatenate([np.repeat(np.arange(keys) - 2, rows), rng.integers(1000, 9000, 700)]).astype(np.int32)
    if rows % 2:
        rng.shuffle(rk)
    sk = np.concatenate([np.arange(-4, keys), rng.integers(1000, 9000, 900)]).astype(np.int32)
    check(rk, sk, PLANS[plan], one_pass, keys)


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("plan", range(len(PLANS)))
@pytest.mark.parametrize("n_r,others", [(4096, 0), (4097, 0), (8191, 1), (70000, 65000), (140001, 100)])
def test_heavy_tuples(n_r, others, plan, one_pass):
    """Five S tuples, three with one key, meet keys of many rows; the last R row is one of them."""
    rng = np.random.default_rng(n_r + others)
    rk = np.full(n_r, 64, dtype=np.int32)
    rk[:others] = rng.integers(0, 1 << 20, others) * 2 + 1
    rk[: n_r // 3: 2] = 96
    rk = rk[rng.permutation(n_r)] if others else rk
    rk[-1] = 64
    check(rk, np.array([64, 96, 7, 64, 64, 96], dtype=np.int32), PLANS[plan], one_pass, n_r)
