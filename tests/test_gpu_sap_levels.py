"""SAP rows projected side by side: strings cut into batches whose rows go level by level.

Bar: as in the other SAP tests, 1e-5 of max|x| plus 1e-6 against the binary64 oracle (a
few row updates per column, each rounded once to binary32).  A row projected beside one
it shares a column with would be off by the size of an update, some 0.01 and more.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_2108_12369_amd import pct
    pct.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pct


def _system(seed, n, m, share):
    """Rows of 1 to 900 distinct columns; a row takes a few columns of an earlier one of the
    last 20 rows with probability `share`, and otherwise lies in a stretch of its own."""
    rng = np.random.default_rng(seed)
    lens = np.where(rng.uniform(size=m) < 0.9, rng.integers(1, 200, m), rng.integers(200, 901, m))
    cols = []
    for i, k in enumerate(int(v) for v in lens):
        start = (i * 997) % (n - 1000)
        c = start + rng.choice(1000, k, replace=False)
        if i and rng.uniform() < share:
            old = cols[int(rng.integers(max(0, i - 20), i))]
            take = min(len(old), k, 3)
            c = np.unique(np.concatenate([c[: k - take], rng.choice(old, take, replace=False)]))
        cols.append(rng.permutation(c))
    rp = np.zeros(m + 1, np.int64)
    rp[1:] = np.cumsum([len(c) for c in cols])
    cols = np.concatenate(cols).astype(np.int32)
    vals = rng.uniform(0.05, 2.0, int(rp[-1])).astype(np.float32)
    b = np.add.reduceat(vals.astype(np.float64) * rng.uniform(0.0, 1.5, n)[cols], rp[:-1]).astype(np.float32)
    return dict(row_ptr=rp, cols=cols, vals=vals, b=b), rng.uniform(0.0, 1.5, n), rng


def _dev(s, *names):
    return [torch.as_tensor(s[k], device="cuda") for k in names]


# rows per string around the batch sizes of 8 and 16; n in LDS, in the workspace, and past
# the columns that one pass of the conflict table takes (162,816)
@pytest.mark.parametrize("n", [20000, 50000, 170000])
@pytest.mark.parametrize("m,M", [(1, 1), (7, 1), (8, 1), (17, 1), (31, 2), (129, 4), (1025, 1), (700, 9)])
@pytest.mark.parametrize("share", [0.0, 0.3, 1.0])
def test_levels(P, oracle, n, m, M, share):
    s, x0, rng = _system(n + 31 * m + M, n, m, share)
    for order in (None, rng.permutation(m)):
        S = P.Sap(*_dev(s, "row_ptr", "cols", "vals", "b"), n, n_strings=M, relax=0.9,
                  order=None if order is None else torch.as_tensor(order, device="cuda"))
        x = torch.as_tensor(x0.astype(np.float32), device="cuda")
        S.iterate(x, 2)
        assert S.status() == 0
        want = oracle.sap(s["row_ptr"], s["cols"], s["vals"].astype(np.float64), s["b"].astype(np.float64), n,
                          x0.astype(np.float32).astype(np.float64), n_iter=2, n_strings=M, relax=0.9, order=order)
        err = float(np.abs(x.cpu().numpy() - want).max())
        assert err <= 1e-5 * float(np.abs(want).max()) + 1e-6, (err, order is None)


@pytest.mark.parametrize("n", [20000, 50000])
def test_order_buffer_changed_between_iterations(P, oracle, n):
    """The levels follow what the order buffer holds when iterate is called."""
    m = 200
    s, x0, rng = _system(n + 5, n, m, 0.7)
    first, then = rng.permutation(m), rng.permutation(m)
    order = torch.as_tensor(first, device="cuda")
    S = P.Sap(*_dev(s, "row_ptr", "cols", "vals", "b"), n, n_strings=3, relax=0.9, order=order)
    x = torch.as_tensor(x0.astype(np.float32), device="cuda")
    want = x0.astype(np.float32).astype(np.float64)
    for o in (first, then):
        order.copy_(torch.as_tensor(o))
        S.iterate(x, 1)
        want = oracle.sap(s["row_ptr"], s["cols"], s["vals"].astype(np.float64), s["b"].astype(np.float64), n, want,
                          n_iter=1, n_strings=3, relax=0.9, order=o)
    err = float(np.abs(x.cpu().numpy() - want).max())
    assert err <= 1e-5 * float(np.abs(want).max()) + 1e-6, err


# y in strips of the grid the columns come from: the row length found among the entries
# (8 grid rows fit n, or not; the last strip cut off by n), several candidates, none
@pytest.mark.parametrize("n,s", [(40904, 5113), (40904, 5114), (50000, 250), (50001, 333), (65536, 2), (50000, 1)])
def test_strip_order(P, oracle, n, s):
    m = 400
    rng = np.random.default_rng(n + s)
    rp, cols = [0], []
    for i in range(m):
        k = int(rng.integers(1, 900))
        c = int(rng.integers(0, n)) + np.cumsum(np.where(rng.uniform(size=k) < 0.5, 1, s) * (1 if i % 2 else -1))
        c = np.unique(c[(c >= 0) & (c < n)])
        cols.append(c)
        rp.append(rp[-1] + len(c))
    rp, cols = np.asarray(rp, np.int64), np.concatenate(cols).astype(np.int32)
    vals = rng.uniform(0.05, 2.0, int(rp[-1])).astype(np.float32)
    xt = rng.uniform(0.0, 1.5, n)
    b = np.bincount(np.repeat(np.arange(m), np.diff(rp)), vals.astype(np.float64) * xt[cols], minlength=m).astype(np.float32)
    S = P.Sap(*(torch.as_tensor(v, device="cuda") for v in (rp, cols, vals, b)), n, n_strings=7, relax=0.8)
    x = torch.zeros(n, device="cuda")
    S.iterate(x, 2)
    assert S.status() == 0
    want = oracle.sap(rp, cols, vals.astype(np.float64), b.astype(np.float64), n, np.zeros(n), n_iter=2, n_strings=7,
                      relax=0.8)
    err = float(np.abs(x.cpu().numpy() - want).max())
    assert err <= 1e-5 * float(np.abs(want).max()) + 1e-6, err
