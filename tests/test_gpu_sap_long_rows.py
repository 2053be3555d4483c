"""SAP with y in the workspace: rows prepared and levelled in one pass, rows past a slot.

Row lengths lie around the chunks that are kept in registers (512 entries), the staged slot
(768), four more chunks of it (1024) and the longest row whose columns are compared (4096).
Bar: as in the other SAP tests, 1e-5 of max|x| plus 1e-6 against the binary64 oracle.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N = 50001
LENS = [1, 2, 63, 64, 65, 511, 512, 513, 767, 768, 769, 1023, 1024, 1025, 1279, 1281, 4095, 4096, 4097, 0]


@pytest.fixture(scope="module")
def P():
    from paper_2108_12369_amd import pct
    pct.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pct


def _system(seed, m, repeats, table):
    """m rows of the lengths above; with `repeats`, every third has some columns twice or more;
    with `table`, the columns of a row agree in their low 14 bits by threes."""
    rng = np.random.default_rng(seed)
    rows = []
    for i in range(m):
        k = LENS[int(rng.integers(len(LENS)))]
        c = rng.choice(N // 3, k, replace=False)
        if table:
            c = (c // 3 + (c % 3) * 16384)
        if repeats and i % 3 == 0 and k > 1:
            c[rng.integers(0, k, 1 + k // 50)] = c[0]
        rows.append(rng.permutation(c))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int64)
    cols = np.concatenate(rows).astype(np.int32)
    vals = rng.uniform(0.05, 2.0, int(rp[-1])).astype(np.float16)
    xt = rng.uniform(0.0, 1.5, N)
    b = np.bincount(np.repeat(np.arange(m), np.diff(rp)), vals.astype(np.float64) * xt[cols], minlength=m)
    return rp, cols, vals, b.astype(np.float32)


@pytest.mark.parametrize("m,M", [(16, 1), (33, 2), (150, 9)])
@pytest.mark.parametrize("repeats", [False, True])
@pytest.mark.parametrize("table", [False, True])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_long_rows(P, oracle, m, M, repeats, table, dtype):
    rp, cols, vals, b = _system(m + repeats + 2 * table, m, repeats, table)
    S = P.Sap(*(torch.as_tensor(v, device="cuda") for v in (rp, cols)), torch.as_tensor(vals, device="cuda").to(dtype),
              torch.as_tensor(b, device="cuda"), N, n_strings=M, relax=0.8)
    x = torch.zeros(N, device="cuda")
    S.iterate(x, 2)
    assert S.status() == 0
    want = oracle.sap(rp, cols, vals.astype(np.float64), b.astype(np.float64), N, np.zeros(N), n_iter=2, n_strings=M,
                      relax=0.8)
    err = float(np.abs(x.cpu().numpy() - want).max())
    assert err <= 1e-5 * float(np.abs(want).max()) + 1e-6, err


@pytest.mark.parametrize("where", [0, 600, 4100])
@pytest.mark.parametrize("bad", [-1, N])
def test_bad_column(P, where, bad):
    m, k = 20, 4200
    cols = np.tile(np.arange(k, dtype=np.int32), (m, 1))
    cols[13, where] = bad
    args = [torch.as_tensor(v, device="cuda") for v in (np.arange(m + 1, dtype=np.int64) * k, cols.reshape(-1),
                                                        np.ones(m * k, np.float32), np.ones(m, np.float32))]
    S = P.Sap(*args, N, n_strings=1, relax=0.8)
    assert S.status() == P.PCT_EINVAL


@pytest.mark.parametrize("n", [20000, N])
@pytest.mark.parametrize("m,M", [(1, 1), (7, 7), (200, 3), (150, 140)])
def test_prepared_with_an_order_iterated_without(P, oracle, n, m, M):
    """The coefficients are per row: a prepare with an order serves an iterate in natural order."""
    rng = np.random.default_rng(m + n)
    lens = rng.integers(1, 300, m)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    cols = np.concatenate([rng.choice(2000, k, replace=False) for k in lens]).astype(np.int32)
    vals = rng.uniform(0.05, 2.0, int(rp[-1])).astype(np.float32)
    b = np.add.reduceat(vals.astype(np.float64) * rng.uniform(0.0, 1.5, n)[cols], rp[:-1]).astype(np.float32)
    S = P.Sap(*(torch.as_tensor(v, device="cuda") for v in (rp, cols, vals, b)), n, n_strings=M, relax=0.8,
              order=torch.as_tensor(rng.permutation(m), device="cuda"))
    S.p.order_dev = None
    x = torch.zeros(n, device="cuda")
    S.iterate(x, 2)
    assert S.status() == 0
    want = oracle.sap(rp, cols, vals.astype(np.float64), b.astype(np.float64), n, np.zeros(n), n_iter=2, n_strings=M,
                      relax=0.8)
    err = float(np.abs(x.cpu().numpy() - want).max())
    assert err <= 1e-5 * float(np.abs(want).max()) + 1e-6, err
