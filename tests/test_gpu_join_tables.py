"""GPU parity of the join kernels' tables at their edges: LDS tables filled to the last row
and one row less or more (the HBM table), keys that differ only in their lowest or highest
free bits, long chains of one key, S chunks that end at a probe round or a tuple past it;
HBM tables of one or of many partitions beside LDS ones, and past the sizes from which
heavy S tuples are queued.  Integer results: exact equality."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_1307_1955_amd.hj as hj  # noqa: E402

DEV = torch.device("cuda:0")


def check(p, rk, sk):
    rk, sk = np.asarray(rk).astype(np.int32), np.asarray(sk).astype(np.int32)
    rng = np.random.default_rng(len(rk))
    rk, sk = rk[rng.permutation(len(rk))], sk[rng.permutation(len(sk))]
    rr, sr = np.arange(len(rk), dtype=np.int32) * 3 + 1, np.arange(len(sk), dtype=np.int32) - 7
    want = oracle.canonical(*oracle.join(rk, rr, sk, sr))
    t = [torch.from_numpy(a).to(DEV) for a in (rk, rr, sk, sr)]
    o_r, o_s, cnt = hj.join(*t, p=p, capacity=len(want) + 5)
    assert cnt == len(want)
    assert np.array_equal(oracle.canonical(o_r.cpu().numpy()[:cnt], o_s.cpu().numpy()[:cnt]), want)


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("hash", ["identity", "murmur2"])
@pytest.mark.parametrize("lds_cap,bits", [(256, (1,)), (2048, (2,)), (2560, (1, 2)), (4416, (4,)), (8192, (1,)), (8192, (2, 9))])
def test_lds_table_edges(lds_cap, bits, hash, one_pass):
    B = sum(bits)
    P = 1 << B
    p = hj.params("phj", len(bits), bits, hash=hash, lds_cap=lds_cap, one_pass=one_pass)
    # identity: partition i takes keys i mod P; three partitions get cap - 1, cap and cap + 1 rows
    rows = [lds_cap - 1, lds_cap, lds_cap + 1]
    rk = np.concatenate([np.arange(n, dtype=np.int64) * P + i % P for i, n in enumerate(rows[: min(3, P)])])
    rk = np.concatenate([rk, np.full(70, rk[0]), rk[:3] ^ 0x80000000, [-(2 ** 31), 2 ** 31 - 1]])
    sk = np.concatenate([rk[::3], rk[:5], rk[: 2 * 4608 + 1] + P, np.full(600, rk[1])])
    check(p, rk & 0xFFFFFFFF, sk & 0xFFFFFFFF)


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("n_s", [4608, 9217, 40001])
@pytest.mark.parametrize("n_r,heavy,bits,lds_cap", [
    (3000, 0, (2,), 256),            # every partition has an HBM table
    (20000, 700, (6,), 512),         # one of 64
    (200000, 0, (3,), 256),          # more build items than workgroups of the join
    (90000, 70000, (2,), 4416),      # queued heavy tuples (one-pass), 2 x 2^16 rows
    (150000, 140000, (1, 3), 4416),
])
def test_hbm_tables(n_r, heavy, bits, lds_cap, n_s, one_pass):
    rng = np.random.default_rng(n_r + n_s)
    rk = rng.permutation(n_r) + 1
    rk[:heavy] = 77
    sk = rng.integers(1, 2 * n_r, size=n_s)
    sk[:9] = 77
    check(hj.params("phj", len(bits), bits, lds_cap=lds_cap, one_pass=one_pass), rk, sk)
