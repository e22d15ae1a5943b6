"""GPU parity where the partitioning changes its route (csrc/hj_internal.h): starts summed
by the scatter or by a launch of their own, one or eight cursors per partition, tiles of
16384 tuples, one scatter or two, final partitions counted by the one histogram or by a
second one, HBM tables cleared by the scatter.  Integer results: exact equality."""
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

# (|R|, |S|, params): the sizes on both sides of each rule
ROUTES = [
    # starts summed by the scatter: one tile, a tuple more, fewer than a 16-byte chunk, one bit
    (4096, 4096, dict(passes=1, bits=(6,))),
    (4097, 8193, dict(passes=1, bits=(8,))),
    (3, 1, dict(passes=1, bits=(1,))),
    (2, 40001, dict(passes=2, bits=(1, 1), lds_cap=256)),
    (30011, 90017, dict(passes=1, bits=(2,), lds_cap=256, tile=1024)),  # cleared by R's tiles
    # 64 tiles x 2^8 counts are the last that the scatter sums; one tile more, and 64 tiles have 8 cursors
    (32 * 1024, 32 * 1024, dict(passes=1, bits=(8,), tile=1024)),
    (32 * 1024 + 1, 32 * 1024, dict(passes=1, bits=(8,), tile=1024)),
    (63 * 1024 - 5, 1024, dict(passes=1, bits=(9,), tile=1024)),
    (200001, 30, dict(passes=1, bits=(1,), lds_cap=256, tile=1024)),   # starts launch with 2 partitions
    (64 * 2048, 2048 * 70 - 3, dict(passes=2, bits=(3, 7), tile=2048, lds_cap=256)),
    # 16384-tuple tiles from 256 of them on (12 bits); the last is partial
    (1 << 21, (1 << 21) + 1, dict(passes=2, bits=(6, 6))),
    ((1 << 21) - 1, 1 << 21, dict(passes=1, bits=(12,), hash="murmur2")),
    (1 << 21, 1 << 21, dict(passes=1, bits=(13,), tile=8192)),
    # two scatters: counted by the one histogram from 400 tuples per partition on, else by a second one
    (400000, 160 * 8192 - 400000, dict(passes=2, bits=(7, 6))),
    (400000, 160 * 8192 - 400001, dict(passes=2, bits=(7, 6))),
    (1 << 20, 2 << 20, dict(passes=2, bits=(7, 7), lds_cap=256, hash="murmur2")),
    (1 << 20, 5 << 20, dict(passes=2, bits=(3, 12))),
    (1 << 20, 1 << 20, dict(passes=2, bits=(9, 6), lds_cap=256)),
    (1400000, 400 * 8192 - 1400000, dict(passes=2, bits=(7, 6))),  # the line between the two
    (1400000, 400 * 8192 - 1400001, dict(passes=2, bits=(7, 6))),
    (1 << 20, 12 << 20, dict(passes=2, bits=(3, 12))),
    (500009, 700001, dict(passes=2, bits=(8, 8))),
]


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("case", range(len(ROUTES)))
def test_routes(case, one_pass):
    n_r, n_s, kw = ROUTES[case]
    r, s = gen.unique_uniform(60 + case, n_r, n_s, 2 * n_r)
    rk = r.key.copy()
    rk[: n_r // 8] = rk[n_r // 8: n_r // 8 * 2]  # an eighth of the keys twice
    t = [torch.from_numpy(a).to(DEV) for a in (rk, r.rid, s.key, s.rid)]
    o_r, o_s, cnt = hj.join(*t, p=hj.params("phj", one_pass=one_pass, **kw), capacity=2 * n_s)
    want = oracle.canonical(*oracle.join(rk, r.rid, s.key, s.rid))
    assert cnt == len(want)
    assert np.array_equal(oracle.canonical(o_r.cpu().numpy(), o_s.cpu().numpy()), want)


@pytest.mark.parametrize("n_r,n_s,bits", [(20000, 3000, (4,)), (20000, 3000, (3, 4)), (1 << 20, 300001, (2, 5))])
def test_probe_clears_tables_of_a_built_table(n_r, n_s, bits):
    """Oversized partitions of a built R: the probe's scatter clears their tables in its own
    workspace, which holds another call's words before each probe."""
    r, s = gen.unique_uniform(90, n_r, n_s, 2 * n_r)
    t = [torch.from_numpy(a).to(DEV) for a in (r.key, r.rid, s.key, s.rid)]
    tab = hj.Table(t[0], t[1], hj.params("phj", len(bits), bits, lds_cap=256, one_pass=True))
    ws = tab.probe_workspace(n_s)
    out = [torch.empty(n_s, dtype=torch.int32, device=DEV) for _ in range(2)]
    d = torch.zeros(1, dtype=torch.int64, device=DEV)
    want = oracle.canonical(*oracle.join(r.key, r.rid, s.key, s.rid))
    for fill in (0, 0x5A, 0xFF):
        ws.fill_(fill)
        hj.hj_probe(tab.t, t[2], t[3], *out, ws, d)
        c = int(d.item())
        assert np.array_equal(oracle.canonical(out[0][:c].cpu().numpy(), out[1][:c].cpu().numpy()), want)
