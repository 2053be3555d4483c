"""SAP iterations with and without a row order, one after another on one workspace.

Bar: as in the other SAP tests, 1e-5 of max|x| plus 1e-6 against the binary64 oracle (rows
projected beside ones they share a column with would lose updates of some 0.01).
"""
import ctypes as C

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


def _system(n, m, seed):
    """Neighbouring rows share no column, rows two apart share all: the levels of the natural
    order do not serve another one, nor the other way round."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(100, 300, m)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    cols = np.concatenate([rng.choice(300, k, replace=False) + 300 * (i % 2) for i, k in enumerate(lens)]).astype(np.int32)
    vals = rng.uniform(0.05, 2.0, int(rp[-1])).astype(np.float32)
    xt = rng.uniform(0.0, 1.5, n)
    b = np.add.reduceat(vals.astype(np.float64) * xt[cols], rp[:-1]).astype(np.float32)
    return rp, cols, vals, b


# y in LDS and in the workspace; strings of one row, around a batch, of many
@pytest.mark.parametrize("n", [20000, 50001])
@pytest.mark.parametrize("m,M", [(9, 1), (40, 40), (150, 7)])
@pytest.mark.parametrize("calls", ["non", "oon", "nono", "onno"])
def test_order_given_and_not_given(P, oracle, n, m, M, calls):
    """The first letter is the prepare call, the others iterate calls; o: with an order."""
    rp, cols, vals, b = _system(n, m, m + M)
    order = np.concatenate([np.arange(0, m, 2), np.arange(1, m, 2)])   # rows that share columns side by side
    dev = torch.as_tensor(order, device="cuda")
    given = {"o": dev.data_ptr(), "n": None}
    S = P.Sap(*(torch.as_tensor(v, device="cuda") for v in (rp, cols, vals, b)), n, n_strings=M, relax=0.8,
              order=dev if calls[0] == "o" else None)
    x = torch.zeros(n, device="cuda")
    want = np.zeros(n)
    for c in calls[1:]:
        S.p.order_dev = C.c_void_p(given[c])
        S.iterate(x, 1)
        want = oracle.sap(rp, cols, vals.astype(np.float64), b.astype(np.float64), n, want, n_iter=1, n_strings=M,
                          relax=0.8, order=order if c == "o" else None)
    assert S.status() == 0
    err = float(np.abs(x.cpu().numpy() - want).max())
    assert err <= 1e-5 * float(np.abs(want).max()) + 1e-6, err
