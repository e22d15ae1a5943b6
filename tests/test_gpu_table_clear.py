"""GPU parity where a scatter clears the HBM tables of R's oversized partitions: the second
scatter of a counted plan, and workgroups that only clear, when few tuples probe a large table.
The workspace holds words that are no empty slots before every call."""
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
FILLS = (0x00, 0x5A)


def relations(seed, n_r, n_s, heavy):
    """Unique keys but for one that `heavy` rows of R hold (and about 1 in 2 n_r of S)."""
    r, s = gen.unique_uniform(seed, n_r, n_s, 2 * n_r)
    rk = r.key.copy()
    rk[:heavy] = s.key[n_s // 2]
    return (rk, r.rid, s.key, s.rid), [torch.from_numpy(a).to(DEV) for a in (rk, r.rid, s.key, s.rid)]


def check(out, d, want):
    c = int(d.item())
    assert c == len(want)
    assert np.array_equal(oracle.canonical(out[0][:c].cpu().numpy(), out[1][:c].cpu().numpy()), want)


def result_columns(n):
    return [torch.empty(n, dtype=torch.int32, device=DEV) for _ in range(2)], torch.zeros(1, dtype=torch.int64, device=DEV)


# two scatters, counted by the one histogram (13 bits from 400 tuples a partition on); only the
# heavy key's partition is larger than lds_cap, or all are (12 bits: the scatter of one pass)
JOINS = [(400000, 3000000, (7, 6), 5000), (400000, 3000000, (8, 5), 300), (1 << 20, 1 << 20, (6, 6), 0),
         (3400000, 40000, (7, 6), 0)]


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("case", range(len(JOINS)))
def test_join_clears_tables(case, one_pass):
    n_r, n_s, bits, heavy = JOINS[case]
    h, t = relations(70 + case, n_r, n_s, heavy)
    want = oracle.canonical(*oracle.join(*h))
    p = hj.params("phj", 2, bits, lds_cap=256, one_pass=one_pass)
    ws = hj.workspace(p, n_r, n_s)
    out, d = result_columns(len(want) + 1)
    for fill in FILLS:
        ws.fill_(fill)
        hj.hj_join(p, *t, *out, ws, d)
        hj.hj_workspace_status(ws)
        check(out, d, want)


PROBES = [
    # a counted plan's second scatter, the table's partitions instead of R's tuples
    (400000, 3300000, (7, 6), 256, 5000),
    # few tuples: one tile, and up to 256 workgroups that only clear; one S partition, some, all
    (1 << 20, 1, (4,), 0, 0), (1 << 20, 1000, (4,), 256, 0), (1 << 20, 1, (6, 6), 256, 0),
    (1 << 20, 3000, (6, 6), 256, 20000), (4097, 2, (1,), 256, 0), (70001, 9000, (2, 5), 256, 0),
    (1 << 20, 300000, (3, 6), 256, 0),
    # cleared by a launch of its own: not counted, and more than 6 bits in pass 2
    (1 << 20, 1000, (7, 7), 256, 3000),
]


@pytest.mark.parametrize("one_pass", [True, False], ids=["1pass", "2pass"])
@pytest.mark.parametrize("case", range(len(PROBES)))
def test_probe_clears_tables(case, one_pass):
    n_r, n_s, bits, cap, heavy = PROBES[case]
    h, t = relations(80 + case, n_r, n_s, heavy)
    want = oracle.canonical(*oracle.join(*h))
    tab = hj.Table(t[0], t[1], hj.params("phj", len(bits), bits, lds_cap=cap, one_pass=one_pass))
    ws = tab.probe_workspace(n_s)
    out, d = result_columns(len(want) + 1)
    for fill in FILLS:
        ws.fill_(fill)
        hj.hj_probe(tab.t, t[2], t[3], *out, ws, d)
        hj.hj_workspace_status(ws)
        check(out, d, want)
