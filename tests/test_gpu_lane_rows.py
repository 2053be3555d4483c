"""Rows walked one lane each (their spline may leave the grid box), beside and after the
wave walk: every row of a call, a few of its rows, and none; against the oracle with the
bar of tests/parity.py, and the same bits from a persistent grid (another launch of them)."""
import numpy as np
import pytest
import torch

from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_2108_12369_amd import pct
    pct.lib()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pct


def _cfg(W, dim, fit, rows):
    n, h = ((50, 46), (200.0 * fit / 50, 160.0 * fit / 46)) if dim == 2 else \
        ((30, 26, 24), (200.0 * fit / 30, 160.0 * fit / 26, 170.0 * fit / 24))
    ph = W.phantom(dim, n, h, W.neo1_regions() if dim == 2 else W.neo_ellipsoid_regions())
    return W.workload("lane-rows", ph, W.beam(63, 24, 15.0, rows, (-95.0, 95.0), (-80.0, 80.0), noise_rel=0.01,
                                              **W.CURVED), "f32")


# fit: the grid box against the phantom (0.8: most curved rows leave it, 1.0: a few in 3D,
# 1.3: none); rows: below one count tile, a few tiles, and more than 1,024 tiles of 256
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("fit,rows", [(0.8, 200), (0.8, 3001), (0.8, 300_000), (1.0, 300_000), (1.3, 3001)])
def test_lane_rows(P, oracle, W, dim, fit, rows):
    cfg = _cfg(W, dim, fit, rows)
    out = P.simulate(cfg)
    sample = np.unique(np.linspace(0, rows - 1, min(rows, 3000)).astype(np.int64))
    g = parity.gather_rows(out["row_ptr"], out["cols"], out["vals"], out["b"], sample)
    st = parity.compare(g, oracle.run(cfg, rows=sample), min(cfg["phantom"]["h"][:dim]), "f32")
    assert st["n_failures"] == 0, st["failures"][:3]
    try:
        P.set_launch_config(blocks_per_cu=4)
        q = P.simulate(cfg)
    finally:
        P.set_launch_config()
    for k in ("row_ptr", "cols", "vals", "b"):
        assert torch.equal(out[k], q[k]), k
    b = torch.empty(rows, dtype=torch.float32, device="cuda")
    js = P.JobSet()
    js.add(cfg["phantom"], cfg["beam"], out["x"], b=b)
    P.wepl(js, torch.empty(P.workspace_bytes(js), dtype=torch.uint8, device="cuda"))
    assert torch.equal(b, out["b"])
