"""Calls of few rows: fewer rows per wavefront, the same rows.  A row depends on its proton
number alone, so a call over a range of rows gives the bits of the larger call's rows
(tolerance: none)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_2108_12369_amd import pct
    pct.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pct


@pytest.fixture(scope="module", params=["2d-straight", "3d-curved"])
def whole(request, P, W):
    n = 300_000
    if request.param == "2d-straight":
        cfg = W.scaled(W.c_paper(), n_protons=n)
    else:
        ph = W.phantom(3, (64, 60, 48), (3.1, 3.1, 3.4), W.neo_ellipsoid_regions())
        cfg = W.workload("small-batches", ph, W.beam(41, 45, 8.0, n, (-98.0, 98.0), (-80.0, 80.0), noise_rel=0.01,
                                                     **W.CURVED), "f16")
    return cfg, P.simulate(cfg)


# 256 CUs: one row per wave below 32,768 rows, 2 up to 65,536, 4 up to 131,072, then 8
@pytest.mark.parametrize("rows", [1, 3, 255, 4097, 32767, 32768, 65535, 65536, 131071, 131073])
def test_range_of_rows(P, whole, rows):
    cfg, w = whole
    begin = 300_000 - rows - 77
    o = P.simulate(cfg, row_begin=begin, row_count=rows, x=w["x"])
    lo, hi = int(w["row_ptr"][begin]), int(w["row_ptr"][begin + rows])
    assert torch.equal(o["row_ptr"], w["row_ptr"][begin:begin + rows + 1] - lo)
    assert torch.equal(o["cols"], w["cols"][lo:hi])
    assert torch.equal(o["vals"], w["vals"][lo:hi])
    assert torch.equal(o["b"], w["b"][begin:begin + rows])
    b = torch.empty(rows, dtype=torch.float32, device="cuda")
    js = P.JobSet()
    js.add(cfg["phantom"], cfg["beam"], w["x"], b=b, row_begin=begin, row_count=rows)
    P.wepl(js, torch.empty(P.workspace_bytes(js), dtype=torch.uint8, device="cuda"))
    assert torch.equal(b, o["b"])
