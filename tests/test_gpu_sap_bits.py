"""SAP: rows that share no column projected side by side give the bits of the rows projected one
after another, where no row repeats a column.  A prepare with an order leaves the levels of rows
one after another for an iterate without it.  No tolerance.
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


# y in LDS and in the workspace; strings of one row, around a batch, of many; few and many
# columns shared; rows past the chunks in registers
@pytest.mark.parametrize("n", [20000, 50001])
@pytest.mark.parametrize("m,M", [(9, 1), (40, 40), (150, 7), (1500, 20)])
@pytest.mark.parametrize("width", [1000, 19000])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_bits(P, n, m, M, width, dtype):
    rng = np.random.default_rng(n + m + width)
    lens = np.where(rng.uniform(size=m) < 0.95, rng.integers(1, 400, m), rng.integers(400, 1000, m))
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    cols = np.concatenate([rng.choice(width, k, replace=False) for k in lens]).astype(np.int32)
    vals = rng.uniform(0.05, 2.0, int(rp[-1])).astype(np.float16)
    b = np.add.reduceat(vals.astype(np.float64) * rng.uniform(0.0, 1.5, n)[cols], rp[:-1]).astype(np.float32)
    A = [torch.as_tensor(v, device="cuda") for v in (rp, cols, vals, b)]
    A[2] = A[2].to(dtype)
    order = torch.arange(m, device="cuda")
    S = P.Sap(*A, n, n_strings=M, relax=0.9)
    side = S.iterate(torch.zeros(n, device="cuda"), 3)
    again = S.iterate(torch.zeros(n, device="cuda"), 3)
    T = P.Sap(*A, n, n_strings=M, relax=0.9, order=order)
    ordered = T.iterate(torch.zeros(n, device="cuda"), 3)
    T.p.order_dev = None
    one = T.iterate(torch.zeros(n, device="cuda"), 3)
    assert S.status() == 0 and T.status() == 0 and float(one.abs().max()) > 0.01
    assert torch.equal(side, one) and torch.equal(again, one) and torch.equal(ordered, one)
