"""Row offsets: summed by the blocks that write row_ptr, or scanned first when a call has more
tiles of 256 rows than that pays for (jobs of n tiles with n^2 summing to 2^24).  Whole
numbers: no tolerance."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LIMIT = 4096 * 256


@pytest.fixture(scope="module")
def P():
    from paper_2108_12369_amd import pct
    pct.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pct


def _count(P, cfg, x, ranges, precision):
    js, rps = P.JobSet(), []
    cols = torch.empty(1, dtype=torch.int32, device="cuda")
    vals = torch.empty(1, dtype=torch.float16, device="cuda")
    b = torch.empty(1, dtype=torch.float32, device="cuda")
    for begin, rows in ranges:
        rps.append(torch.full((rows + 1,), -1, dtype=torch.int64, device="cuda"))
        js.add(cfg["phantom"], cfg["beam"], x, row_ptr=rps[-1], cols=cols, vals=vals, nnz_capacity=1, b=b,
               row_begin=begin, row_count=rows, precision=precision)
    ws = torch.empty(P.workspace_bytes(js), dtype=torch.uint8, device="cuda")
    total = torch.full((len(ranges),), -1, dtype=torch.int64, device="cuda")
    P.count_rows(js, ws, total)
    return rps, total


@pytest.mark.parametrize("precision", ["mixed", "plain_f32"])
def test_offsets(P, W, precision):
    cfg = W.scaled(W.c_paper(), n_protons=LIMIT + 257)
    x = P.phantom_build(cfg["phantom"])
    (want,), total = _count(P, cfg, x, [(0, LIMIT + 257)], precision)       # scanned
    assert int(total[0]) == int(want[-1]) and int(want[0]) == 0 and bool((want[1:] >= want[:-1]).all())
    for ranges in ([(0, LIMIT)], [(1, LIMIT)], [(0, LIMIT - 1)], [(0, LIMIT + 1)], [(3, 1)], [(5, 256)], [(5, 257)],
                   # jobs without a tile; more jobs than one launch's arguments hold
                   [(9, 0), (0, 300), (4, 0), (4, 0), (7, 255), (100, 0)],
                   [(17 * k, 1 + (k * 7919) % 3000) for k in range(40)],
                   [(0, LIMIT // 4)] * 16, [(0, LIMIT // 4)] * 17):
        rps, total = _count(P, cfg, x, ranges, precision)
        for k, (begin, rows) in enumerate(ranges):
            assert torch.equal(rps[k], want[begin:begin + rows + 1] - want[begin]), (k, begin, rows)
            assert int(total[k]) == int(want[begin + rows] - want[begin])
