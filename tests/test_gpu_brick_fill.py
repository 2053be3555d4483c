"""The bricked copy of x that the b gathers read: grids whose rows are not whole bricks or whole
float4, x at an address that is only a float's.  pct_wepl_static reads x itself, so b must have
the same bits (tolerance: none)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_2108_12369_amd import pct
    pct.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pct


@pytest.mark.parametrize("n", [(1, 9, 3), (2, 8, 5), (3, 7, 4), (4, 5, 1), (5, 17, 6), (6, 16, 2), (7, 8, 2), (8, 8, 8),
                               (9, 9, 9), (13, 21, 11), (64, 1, 3), (131, 66, 40), (200, 200, 33)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_bricks(P, W, n, offset):
    g = torch.Generator(device="cuda")
    g.manual_seed(n[0])
    nv = n[0] * n[1] * n[2]
    x = torch.rand(nv + offset, device="cuda", generator=g)[offset:]
    ph = W.phantom(3, n, (1.0, 1.1, 0.9), W.neo_ellipsoid_regions())
    got = []
    for static in (False, True):
        js, bs = P.JobSet(), []
        for kw in ({}, W.CURVED):
            half = 0.6 * max(n[0], n[1])
            bm = W.beam(5, 12, 15.0, 1500, (-half, half), (-0.6 * n[2], 0.6 * n[2]), **kw)
            bs.append(torch.full((1500,), -1.0, device="cuda"))
            js.add(ph, bm, x, b=bs[-1])
        if static:
            status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
            P.wepl_static(js, status)
            assert int(status) == 0
        else:
            ws = torch.empty(P.workspace_bytes(js), dtype=torch.uint8, device="cuda").fill_(0xff)
            P.wepl(js, ws)
            assert P.device_status(ws) == 0
        got.append(torch.cat(bs))
    assert bool((got[1] > 0).any())
    assert torch.equal(got[0], got[1])
