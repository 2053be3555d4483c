"""The weighted-area rule for regions that are tiny against their coordinates, where the rounding
of a sample point is a visible part of the region: against the oracle, bit for bit (the same
points, the same tests and sums that binary64 holds exactly)."""
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


@pytest.mark.parametrize("angle", [0.0, 30.0])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("at", [1e3, 1e6, 1e12])
def test_area_far_and_tiny(P, oracle, W, dim, at, angle):
    n, S = ((45, 45), 64) if dim == 2 else ((23, 23, 9), 16)
    h = 0.05 if at > 1e9 else 5e-7 * 45 / n[0]
    c = (at, 2.0 * at, 0.5 * at)[:dim]
    semi = [v * h * n[0] for v in (0.4, 0.3, 0.2)][:dim]
    kind = "ellipse" if dim == 2 else "ellipsoid"
    ph = W.phantom(dim, n, (h,) * dim, [W._e(c, semi, 1.25, kind, angle_deg=angle),
                                        W._e(c, [0.5 * v for v in semi], 0.75, kind, angle_deg=-angle)],
                   voxelize="area_avg", area_samples=S)
    ph["origin"] = [c[d] - 0.5 * n[d] * h for d in range(dim)]
    assert np.array_equal(P.phantom_build(ph).cpu().numpy(), oracle.phantom_build(ph))
