"""Rows of 1 to 1023 entries written from the wave's LDS slice, in groups of 3, 4 and 5 times
64 entries: straight rows of every length around the group limits on long narrow grids, packed
coordinates and plain columns, with and without A, constant chords; against the oracle (bar of
tests/parity.py)."""
import numpy as np
import pytest
import torch

from tests import parity

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 63, 64, 65, 128, 129, 191, 192, 193, 256, 257, 320, 321, 384, 385, 448, 449, 512, 513, 576, 577, 640, 641,
           704, 768, 832, 896, 960, 977, 978, 979, 1015, 1023]


@pytest.mark.parametrize("dim,path", [(2, "straight"), (3, "straight"), (2, "hermite"), (3, "hermite")])
def test_row_lengths(oracle, W, dim, path):
    from paper_2108_12369_amd import pct as P
    assert torch.cuda.is_available()
    js, keep = P.JobSet(), []
    for k in LENGTHS:
        # k voxels along x, the beam along it with a small spread
        n, h = ((k, 9), (180.0 / k, 20.0)) if dim == 2 else ((k, 7, 5), (180.0 / k, 20.0, 30.0))
        regs = [W._e((0, 0), (88.0, 70.0), 1.3)] if dim == 2 else [W._e((0, 0, 0), (88.0, 60.0, 70.0), 1.3, "ellipsoid")]
        extra = dict(path=path, step=0.5) if path == "hermite" else {}
        cfg = W.workload("rows", W.phantom(dim, n, h, regs),
                         W.beam(900 + k, 2, 180.0, 40, (-69.0, 69.0), (-59.0, 59.0), noise_rel=0.01, **extra), "f32")
        cap = 40 * 1200
        x = P.phantom_build(cfg["phantom"])
        o = dict(row_ptr=torch.empty(41, dtype=torch.int64, device="cuda"), cols=torch.empty(cap, dtype=torch.int32, device="cuda"),
                 vals=torch.empty(cap, dtype=torch.float32, device="cuda"), b=torch.empty(40, dtype=torch.float32, device="cuda"))
        js.add(cfg["phantom"], cfg["beam"], x, nnz_capacity=cap, **o)
        keep.append((cfg, x, o))
    ws = torch.empty(P.workspace_bytes(js), dtype=torch.uint8, device="cuda")
    P.count_rows(js, ws, torch.empty(len(LENGTHS), dtype=torch.int64, device="cuda"))
    P.emit_csr(js, ws)
    assert P.device_status(ws) == 0
    rows = np.arange(40, dtype=np.int64)
    for k, (cfg, x, o) in zip(LENGTHS, keep):
        g = parity.gather_rows(o["row_ptr"], o["cols"], o["vals"], o["b"], rows)
        st = parity.compare(g, oracle.run(cfg, rows=rows, x=x.cpu().numpy()), min(cfg["phantom"]["h"][:dim]), "f32")
        assert st["n_failures"] == 0, (k, st["failures"][:3])
        assert int((o["row_ptr"][1:] - o["row_ptr"][:-1]).max()) >= k
