"""The autotuner on batches so small that 16, 32 and 64 rows per wave are run alike: it keeps the
largest, not whichever of the equals was timed fastest."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_equal_settings_are_not_told_apart(W):
    from paper_2108_12369_amd import pct as P
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ph = W.phantom(2, (64, 64), (3.0, 3.0), W.neo1_regions())
    try:
        P.autotune_cache_clear()
        for rows in (200, 500, 1100, 3000, 9000, 30000):   # a cache key each
            bm = W.beam(3, 10, 36.0, rows, (-95.0, 95.0))
            out = P.simulate(W.workload("small", ph, bm))
            js = P.JobSet()
            js.add(ph, bm, out["x"], row_ptr=out["row_ptr"], cols=out["cols"], vals=out["vals"], b=out["b"],
                   nnz_capacity=out["nnz"])
            ws = torch.empty(P.workspace_bytes(js), dtype=torch.uint8, device="cuda")
            best = P.autotune(js, ws, torch.empty(1, dtype=torch.int64, device="cuda"))
            assert best["rows_per_wave"] == 64, (rows, best)
            assert P.autotune_cached(js) == best
    finally:
        P.autotune_cache_clear()
        P.set_launch_config()
