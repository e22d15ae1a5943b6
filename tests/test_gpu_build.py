"""GPU parity of the chained-table builds (SHJ, and the HBM tables of oversized PHJ
partitions) where the lanes of a wave share keys: one key only, runs of 2 to 65 rows, a
heavy key among unique or duplicate ones, and ends of rows off the wave and block sizes.
Integer results: exact equality."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1307_1955_amd.hj as hj  # noqa: E402

DEV = torch.device("cuda:0")


def one_key(n, rng):
    return np.full(n, 5)


def two_keys(n, rng):
    return np.arange(n) % 2


def sorted_runs(n, rng):
    return np.repeat(np.arange(n), rng.choice([1, 2, 63, 64, 65], size=n))[:n]


def heavy_among_unique(n, rng):  # a key too rare for two rows of most waves
    k = np.arange(n) + 10
    k[rng.random(n) < 0.02] = 3
    return k


def heavy_among_duplicates(n, rng):
    k = rng.integers(10, 10 + max(1, n // 4), size=n)
    k[rng.random(n) < 0.2] = -(2 ** 31)
    return k


KINDS = [one_key, two_keys, sorted_runs, heavy_among_unique, heavy_among_duplicates]


@pytest.mark.parametrize("n_r", [1, 65, 2049, 300007])
@pytest.mark.parametrize("kind", KINDS, ids=[k.__name__ for k in KINDS])
def test_shared_keys(kind, n_r):
    rng = np.random.default_rng(n_r)
    rk = kind(n_r, rng).astype(np.int32)
    sk = np.unique(rk)
    sk = np.concatenate([sk[rng.permutation(len(sk))[:4096]], [2, 2 ** 31 - 1]]).astype(np.int32)
    rr, sr = np.arange(n_r, dtype=np.int32) * 3 + 1, np.arange(len(sk), dtype=np.int32) - 7
    t = [torch.from_numpy(a).to(DEV) for a in (rk, rr, sk, sr)]
    want = oracle.canonical(*oracle.join(rk, rr, sk, sr))
    for p in (hj.params("shj"), hj.params("shj", one_pass=True), hj.params("phj", 1, (1,), lds_cap=256, one_pass=True),
              hj.params("phj", 2, (1, 3), lds_cap=256)):
        o_r, o_s, cnt = hj.join(*t, p=p, capacity=len(want) + 5)
        assert cnt == len(want)
        assert np.array_equal(oracle.canonical(o_r.cpu().numpy()[:cnt], o_s.cpu().numpy()[:cnt]), want)
