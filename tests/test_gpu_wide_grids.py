"""Curved rows on grids whose column strides reach 2^23, where the 24-bit column steps of
the fast item walk end and the general one takes over; against the oracle, bar of
tests/parity.py (columns exact)."""
import numpy as np
import pytest
import torch

from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 23) - 1, 1 << 23])
def test_wide_2d_grid(oracle, W, n):
    from paper_2108_12369_amd import pct as P
    assert torch.cuda.is_available()
    # beams along y on a grid of n x 3 narrow voxels: rows of a few entries whose columns
    # use the full stride; no scattering, so that x stays in one voxel
    ph = W.phantom(2, (n, 3), (80.0 / n, 50.0), [W._e((0, 0), (38.0, 70.0), 1.3)])
    bm = W.beam(77, 2, 180.0, 600, (-37.0, 37.0), path="hermite", step=7.0, angle0_deg=90.0)
    cfg = W.workload("wide", ph, bm, "f32")
    out = P.simulate(cfg)
    rows = np.arange(600, dtype=np.int64)
    g = parity.gather_rows(out["row_ptr"], out["cols"], out["vals"], out["b"], rows)
    st = parity.compare(g, oracle.run(cfg, rows=rows, x=out["x"].cpu().numpy()), 80.0 / n, "f32")
    assert st["n_failures"] == 0, st["failures"][:3]
    assert int(out["cols"].max()) >= 2 * n


@pytest.mark.parametrize("n", [(2896, 2896, 2), (2898, 2896, 2)])
def test_wide_3d_planes(oracle, W, n):
    """Planes of just below and just above 2^23 voxels, on grids too wide for a bricked copy."""
    from paper_2108_12369_amd import pct as P
    assert torch.cuda.is_available()
    ph = W.phantom(3, n, (200.0 / n[0], 200.0 / n[1], 90.0), [W._e((85, 85, 0), (9.0, 9.0, 80.0), 1.3, "ellipsoid")])
    # paths across a corner of the grid, some 800 entries each
    bm = W.beam(78, 1, 360.0, 400, (-127.0, -119.0), (-60.0, 60.0), path="hermite", sigma_in=0.002, sigma_out=0.002,
                sigma_lat=0.2, step=0.05, angle0_deg=135.0)
    cfg = W.workload("wide3", ph, bm, "f32")
    out = P.simulate(cfg)
    rows = np.arange(400, dtype=np.int64)
    g = parity.gather_rows(out["row_ptr"], out["cols"], out["vals"], out["b"], rows)
    st = parity.compare(g, oracle.run(cfg, rows=rows, x=out["x"].cpu().numpy()), 200.0 / n[0], "f32")
    assert st["n_failures"] == 0, st["failures"][:3]
    lens = np.diff(out["row_ptr"].cpu().numpy())
    assert 500 < np.median(lens) and (lens <= 1023).mean() > 0.9
