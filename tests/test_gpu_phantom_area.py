"""The weighted-area rule on the GPU against the oracle, bit for bit: the same points, the
same tests and sums of binary32 values that binary64 holds exactly (tolerance: none)."""
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


def _regions(W, dim):
    if dim == 2:
        return W.neo_turned_regions(25.0, -12.0) + [W._e((7, -9), (0.02, 40.0), 0.7, angle_deg=45.0)]
    regs = W.neo_ellipsoid_regions()
    for r, a in zip(regs, (12.0, 0.0, 30.0, -30.0, 90.0)):
        r["angle_deg"] = a
    return regs + [W._e((0, -40, 0), (15, 5), 1.2, "ellipse", angle_deg=60.0)]   # a turned cylinder


# grids on both sides of a wave (64 voxels) and a block (256); samples on both sides of 64
# points per voxel, and the largest; one voxel larger than every region
@pytest.mark.parametrize("n", [(1, 1), (63, 1), (64, 1), (13, 5), (257, 1), (101, 77)])
@pytest.mark.parametrize("S", [1, 7, 8, 9, 64])
def test_area_2d(P, oracle, W, n, S):
    ph = W.phantom(2, n, (200.0 / n[0], 160.0 / n[1]), _regions(W, 2), voxelize="area_avg", area_samples=S)
    assert np.array_equal(P.phantom_build(ph).cpu().numpy(), oracle.phantom_build(ph))


@pytest.mark.parametrize("n,S", [((1, 1, 1), 13), ((5, 3, 4), 64), ((9, 8, 7), 4), ((33, 17, 11), 3), ((40, 31, 1), 8)])
def test_area_3d(P, oracle, W, n, S):
    ph = W.phantom(3, n, (200.0 / n[0], 160.0 / n[1], 170.0 / n[2]), _regions(W, 3), voxelize="area_avg",
                   area_samples=S)
    assert np.array_equal(P.phantom_build(ph).cpu().numpy(), oracle.phantom_build(ph))


def test_area_points_on_the_boundary(P, oracle, W):
    """Sample points exactly on the boundaries of the regions, and sixteen regions."""
    regs = [W._e((0.0, 0.0), (0.5 * k, 0.5 * k), 0.1 * k) for k in range(16, 0, -1)]
    for S in (1, 3, 5):
        ph = W.phantom(2, (21, 21), (1.0, 1.0), regs, voxelize="area_avg", area_samples=S)
        assert np.array_equal(P.phantom_build(ph).cpu().numpy(), oracle.phantom_build(ph))


def test_area_extreme_axes(P, oracle, W):
    """Semi-axes whose reciprocals overflow or vanish."""
    regs = [W._e((0.0, 0.0), (1e300, 60.0), 1.5), W._e((0.0, 0.0), (1e-310, 40.0), 0.5), W._e((3.0, 0.0), (1e-3, 1e-3), 1.0)]
    ph = W.phantom(2, (21, 21), (6.0, 6.0), regs, voxelize="area_avg", area_samples=3)
    assert np.array_equal(P.phantom_build(ph).cpu().numpy(), oracle.phantom_build(ph))
