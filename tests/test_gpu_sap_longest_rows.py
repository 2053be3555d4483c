"""SAP prepare, rows of more entries than the one-pass prepare names (4,096): whether they repeat a
column is found, so that rows of distinct columns are not projected with atomic adds.

The workspace holds one binary32 coefficient per row from byte 256 on: lambda / ||a_i||^2, negative
for a row that repeats a column.  Bar on its size: 1e-6 of it (binary64 sums rounded once).
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


# columns in one pass of the bitmap (2^19) and in two; the repeated column in the first or the
# last of them, in the row's first and last entries
@pytest.mark.parametrize("n", [50001, 600000])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_repeats_of_long_rows(P, n, dtype):
    rng = np.random.default_rng(n)
    lens = np.resize([4095, 4096, 4097, 5000, 9001, 12288, 3, 4097, 0], 90)
    rows, repeats = [], rng.uniform(size=90) < 0.4
    for i, k in enumerate(lens):
        c = rng.choice(n - 2, k, replace=False) + 1   # columns 0 and n - 1 are kept for repeats
        repeats[i] &= k > 1
        if repeats[i]:
            c[0] = c[-1] = 0 if i % 2 else n - 1
        rows.append(c)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    cols = np.concatenate(rows).astype(np.int32)
    vals = rng.uniform(0.05, 2.0, int(rp[-1])).astype(np.float16)
    dev = [torch.as_tensor(v, device="cuda") for v in (rp, cols, vals, np.ones(90, np.float32))]
    dev[2] = dev[2].to(dtype)
    S = P.Sap(*dev, n, n_strings=5, relax=0.8)
    assert S.status() == 0
    coef = S.ws[256:256 + 4 * 90].view(torch.float32).cpu().numpy().astype(np.float64)
    for i, k in enumerate(lens):
        v = np.bincount(cols[rp[i]:rp[i + 1]], vals[rp[i]:rp[i + 1]].astype(np.float64), minlength=n)
        want = 0.8 / float((v * v).sum()) if k else 0.0
        assert abs(abs(coef[i]) - want) <= 1e-6 * want, (i, k)
        assert (coef[i] < 0) == bool(repeats[i]), (i, k)
