"""The work a user of this framework has it do, as cases of plain values: systems of the
proton-CT simulator (A, b and x), WEPLs alone, phantoms, batches, reconstructions.

A case is a dict with a "kind":
  simulate   the convenience call: phantom, count, emit, outputs allocated by the call
  emit       count_rows and emit_csr into buffers a program keeps (the row chunk of a loop)
  batch      uneven jobs recorded once in one HIP graph, replayed with one launch
  wepl       the WEPLs b alone, without A
  phantom    the voxelised phantom alone
  sap        a reconstruction: prepare, then iterations from zero

exact() traces every path again in binary64 with torch alone, from the paper's formulas
(counter-based draws, boundary solve, cubic Hermite polyline, voxel crossings).
"""
import math

import numpy as np
import torch

from paper_2108_12369_amd import pct
from paper_2108_12369_amd import workloads as W

DEV = "cuda"


# ------------------------------------------------------------------------------ cases
def _grid(dim, nx, ny, nz, h, t, v=0.0, scale=1.0, phantom="neo1"):
    return dict(dim=dim, nx=nx, ny=ny, nz=nz, h=h, t=t, v=v, scale=scale, phantom=phantom)


def _beam(rows, angles, path, dtype, noise=0.0, scatter="fixed", chord=0.0):
    return dict(rows=rows, angles=angles, path=path, dtype=dtype, noise=noise, scatter=scatter, chord=chord)


def listed():
    neo200 = _grid(2, 200, 200, 1, 1.0, 100.0)
    paper = _grid(2, 200, 160, 1, 1.0, 125.0)
    c1 = _grid(2, 400, 400, 1, 0.5, 100.0, phantom="neo2")
    c2 = _grid(3, 200, 200, 160, 1.0, 100.0, 80.0, phantom="ellipsoid")
    c4 = _grid(3, 256, 256, 160, 0.8, 102.4, 64.0, 0.8, phantom="ellipsoid")
    return [
        # the smallest call: a script that looks at a few rows; launches and latency count
        dict(name="simulate-2d-tiny", kind="simulate", **neo200, **_beam(1440, 90, "straight", "f32")),
        # the c0 workload: one ordinary small system, straight paths, FP32 lengths
        dict(name="emit-2d-straight-c0", kind="emit", **neo200, **_beam(92160, 90, "straight", "f32")),
        # the paper's own example: 200 x 160, m = 20 n rows
        dict(name="emit-2d-straight-paper", kind="emit", **paper, **_beam(640000, 180, "straight", "f32")),
        # the c1 workload: a fine 2D grid, curved paths, noise, FP16 lengths
        dict(name="emit-2d-curved-c1", kind="emit", **c1, **_beam(2949120, 360, "hermite", "f16", 0.01)),
        # a 3D job as the 64-job batch draws them, straight paths, an odd number of rows
        dict(name="emit-3d-straight-odd", kind="emit", **_grid(3, 128, 128, 128, 200.0 / 128, 100.0, 100.0, phantom="ellipsoid"),
             **_beam(300001, 77, "straight", "f16", 0.01)),
        # the c2 workload's grid and paths, a tenth of its rows
        dict(name="emit-3d-curved-c2", kind="emit", **c2, **_beam(1000000, 90, "hermite", "f16", 0.01)),
        # the largest: one 5M-row chunk of the head-scale workload c4
        dict(name="emit-3d-curved-c4-chunk", kind="emit", **c4, **_beam(5000000, 180, "hermite", "f16", 0.01)),
        # uneven 2D and 3D jobs, straight and curved, in one graph (the c3 workload's first jobs)
        dict(name="batch-12-jobs-graph", kind="batch", jobs=12, scale=1.0),
        # WEPLs only, for a program that has its own A: curved 3D rows with Highland widths
        dict(name="wepl-3d-curved", kind="wepl", **c2, **_beam(100003, 90, "hermite", "f32", 0.0, "highland")),
        # a phantom by area fractions, turned ellipses, 8 x 8 x 8 points per voxel
        dict(name="phantom-3d-area", kind="phantom", **_grid(3, 160, 160, 128, 1.25, 100.0, phantom="turned"),
             voxelize="area_avg", samples=8),
        # the paper's reconstruction on its example system: 100 strings, iterate in LDS
        dict(name="sap-paper", kind="sap", **paper, **_beam(640000, 180, "straight", "f32"), strings=100, relax=0.1,
             iterations=10),
        # the same on c1's grid with curved rows and FP16 values: the iterate in HBM
        dict(name="sap-2d-curved-400sq", kind="sap", **c1, **_beam(368640, 180, "hermite", "f16", 0.01), strings=100,
             relax=0.1, iterations=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds and ranges."""
    kind = rng.choice(["simulate", "emit", "emit", "emit", "emit", "batch", "wepl", "phantom", "sap", "sap"])
    if kind == "batch":
        return dict(kind=kind, jobs=rng.randint(2, 12), scale=rng.uniform(0.05, 1.0))
    dim = rng.choice([2, 3])
    if kind == "sap":
        dim = 2
    fov = rng.choice([200.0, 204.8, 192.0])
    if dim == 2:
        nx = rng.randint(150, 200) if kind == "sap" and rng.random() < 0.5 else rng.randint(64, 512)
        ny = max(48, int(nx * rng.uniform(0.8, 1.0)))
        g = _grid(2, nx, ny, 1, fov / nx, fov / 2, phantom=rng.choice(["neo1", "neo2", "turned2d"]))
    else:
        nx = rng.randint(64, 256)
        ny = max(64, int(nx * rng.uniform(0.9, 1.0)))
        nz = max(32, int(nx * rng.uniform(0.8, 0.9)))
        g = _grid(3, nx, ny, nz, fov / nx, fov / 2, nz * fov / nx / 2, 0.9, phantom=rng.choice(["ellipsoid", "turned"]))
    if kind == "phantom":
        return dict(kind=kind, **g, voxelize=rng.choice(["area_avg", "corner_avg", "center"]), samples=rng.randint(4, 8))
    path = rng.choice(["straight", "hermite"])
    noise = rng.choice([0.0, rng.uniform(0.0, 0.02)])
    scatter = rng.choice(["fixed", "highland"]) if path == "hermite" else "fixed"
    dtype = rng.choice(["f32", "f16"])
    angles = rng.randint(30, 360)
    if kind == "sap":
        # 12 to 20 equations per unknown, as the paper has it, at most 400,000 rows
        rows = min(400000, int(nx * ny * rng.uniform(12.0, 20.0)))
        return dict(kind=kind, **g, **_beam(rows, angles, path, dtype, noise, scatter), strings=rng.randint(60, 120),
                    relax=rng.choice([0.1, 0.5, 1.0]), iterations=rng.randint(2, 4))
    rows = {"simulate": _log_int(rng, 500, 200000), "emit": _log_int(rng, 10000, 3000000),
            "wepl": _log_int(rng, 1000, 1000000)}[kind]
    chord = g["h"] if kind == "emit" and rng.random() < 0.15 else 0.0
    c = dict(kind=kind, **g, **_beam(rows, angles, path, dtype, noise, scatter, chord))
    # at most the largest listed case's entries
    return dict(c, rows=min(rows, int(rows * 8.0e8 / _size(c))))


# ------------------------------------------------------------------------- descriptors
def _phantom(c):
    dim, s = c["dim"], c["scale"]
    if c["phantom"] == "neo1":
        regs = W.neo1_regions(s, s)
    elif c["phantom"] == "neo2":
        regs = W.neo2_regions()
    elif c["phantom"] == "turned2d":
        regs = W.neo_turned_regions(20.0, 15.0)
    else:
        regs = W.neo_ellipsoid_regions(scale=s)
        if c["phantom"] == "turned":
            for r, a in zip(regs, (15.0, 15.0, 20.0, -20.0, 10.0)):
                r["angle_deg"] = a
    if c["kind"] == "phantom" and dim == 2:
        regs = W.neo_turned_regions(20.0, 15.0)
    n, h = ((c["nx"], c["ny"], c["nz"]), (c["h"],) * 3) if dim == 3 else ((c["nx"], c["ny"]), (c["h"],) * 2)
    return W.phantom(dim, n, h, regs, voxelize=c.get("voxelize", "corner_avg"), area_samples=c.get("samples", 8))


def _make_beam(c, seed):
    extra = dict(W.CURVED) if c["path"] == "hermite" else {}
    return W.beam(seed, c["angles"], 360.0 / c["angles"], c["rows"], (-c["t"], c["t"]), (-c["v"], c["v"]),
                  noise_rel=c["noise"], scatter=c["scatter"], **extra)


def _jobs(c, seed):
    cfgs = W.c3_jobs(n_jobs=c["jobs"])
    for j, cfg in enumerate(cfgs):
        cfg["beam"]["seed"] = seed * 1000 + j
        cfg["beam"]["n_protons"] = max(100, int(cfg["beam"]["n_protons"] * c["scale"]))
    return cfgs


def _config(c, seed):
    return W.workload(c["kind"], _phantom(c), _make_beam(c, seed), c["dtype"], chord_mm=c["chord"] or None)


# ------------------------------------------------------------------- prepare and run
class Buffers:
    """Outputs, workspace and descriptors of a job set; capacities from a bound."""

    def __init__(self, cfgs):
        self.x = [pct.phantom_build(c["phantom"]) for c in cfgs]
        rows = [c["beam"]["n_protons"] for c in cfgs]
        caps = [_capacity(c["phantom"], c["beam"]) for c in cfgs]
        self.row_ptr = [torch.empty(r + 1, dtype=torch.int64, device=DEV) for r in rows]
        self.b = [torch.empty(r, dtype=torch.float32, device=DEV) for r in rows]
        self.cols = [torch.zeros(s, dtype=torch.int32, device=DEV) for s in caps]
        self.vals = [torch.zeros(s, dtype=torch.float16 if c["val_dtype"] == "f16" else torch.float32, device=DEV)
                     for s, c in zip(caps, cfgs)]
        self.nnz = torch.empty(len(cfgs), dtype=torch.int64, device=DEV)
        self.jobs = pct.JobSet()
        for j, c in enumerate(cfgs):
            self.jobs.add(c["phantom"], c["beam"], self.x[j], row_ptr=self.row_ptr[j], cols=self.cols[j],
                          vals=self.vals[j], b=self.b[j], nnz_capacity=caps[j], val_dtype=c["val_dtype"],
                          chord_mm=c["chord_mm"] or 0.0)
        self.ws = torch.empty(pct.workspace_bytes(self.jobs), dtype=torch.uint8, device=DEV)

    def outputs(self):
        return [dict(row_ptr=self.row_ptr[j], cols=self.cols[j], vals=self.vals[j], b=self.b[j], x=self.x[j])
                for j in range(len(self.x))]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "simulate":
        # another seed is another tissue in the same geometry: the system keeps its size
        cfg = _config(case, 7)
        rng = np.random.Generator(np.random.PCG64(seed))
        for r in cfg["phantom"]["regions"]:
            r["rsp"] = round(float(rng.uniform(0.0, 2.0)), 3)
        return dict(kind=kind, cfg=cfg)
    if kind == "phantom":
        ph = _phantom(case)
        rng = np.random.Generator(np.random.PCG64(seed))
        for r in ph["regions"]:
            r["center"] = [v + float(rng.uniform(-2.0, 2.0)) for v in r["center"]]
            r["rsp"] = round(float(rng.uniform(0.0, 2.0)), 3)
        return dict(kind=kind, phantom=ph, x=torch.empty(pct.n_voxels(ph), dtype=torch.float32, device=DEV))
    if kind == "batch":
        buf = Buffers(_jobs(case, seed))
        return dict(kind=kind, buf=buf, graph=pct.Graph(buf.jobs, buf.ws, buf.nnz, build_x=True))
    if kind == "wepl":
        cfg = _config(case, seed)
        x = pct.phantom_build(cfg["phantom"])
        b = torch.empty(case["rows"], dtype=torch.float32, device=DEV)
        js = pct.JobSet()
        js.add(cfg["phantom"], cfg["beam"], x, b=b)
        return dict(kind=kind, jobs=js, x=x, b=b, ws=torch.empty(pct.workspace_bytes(js), dtype=torch.uint8, device=DEV))
    if kind == "sap":
        row_ptr, cols, vals, b, _ = _trace(case, seed, case["dtype"])
        n = case["nx"] * case["ny"]
        return dict(kind=kind, case=case, A=(row_ptr, cols, vals, b), n=n)
    return dict(kind=kind, buf=Buffers([_config(case, seed)]))


def run(state):
    kind = state["kind"]
    if kind == "simulate":
        return pct.simulate(state["cfg"])
    if kind == "phantom":
        return {"x": pct.phantom_build(state["phantom"], state["x"])}
    if kind == "batch":
        state["graph"].launch()
        return {"jobs": state["buf"].outputs(), "nnz": state["buf"].nnz}
    if kind == "wepl":
        pct.wepl(state["jobs"], state["ws"])
        return {"b": state["b"]}
    if kind == "sap":
        c = state["case"]
        solver = pct.Sap(*state["A"], state["n"], n_strings=c["strings"], relax=c["relax"])
        return {"x": solver.iterate(torch.zeros(state["n"], dtype=torch.float32, device=DEV), c["iterations"])}
    buf = state["buf"]
    pct.count_rows(buf.jobs, buf.ws, buf.nnz)
    pct.emit_csr(buf.jobs, buf.ws)
    return {"jobs": buf.outputs(), "nnz": buf.nnz}


# ------------------------------------------------------------------------------- work
def _entries_per_row(dim, n, h, t):
    """Mean number of voxels a straight path crosses, over 64 angles and 256 offsets."""
    phi = (np.arange(64) + 0.5) * (math.pi / 128)
    off = ((np.arange(256) + 0.5) / 128 - 1.0) * t
    c, s = np.cos(phi)[:, None], np.sin(phi)[:, None]
    lo, hi = -np.inf, np.inf
    for q, u, m in ((-off * s, c, n[0] * h / 2), (off * c, s, n[1] * h / 2)):
        lo, hi = np.maximum(lo, (-m - q) / u), np.minimum(hi, (m - q) / u)
    chord = np.maximum(hi - lo, 0.0)
    return float(np.mean((chord > 0) * 1.0 + chord * (c + s) / h))


def _capacity(ph, bm):
    return int(1.05 * bm["n_protons"] * _entries_per_row(ph["dim"], ph["n"], ph["h"][0], bm["t_range"][1])) + 4096


def _size(c):
    return c["rows"] * _entries_per_row(c["dim"], (c["nx"], c["ny"]), c["h"], c["t"])


def work(case):
    kind = case["kind"]
    if kind == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for cfg in _jobs(case, 0):
            ph, bm = cfg["phantom"], cfg["beam"]
            nvox = pct.n_voxels(ph)
            nnz = bm["n_protons"] * _entries_per_row(ph["dim"], ph["n"], ph["h"][0], bm["t_range"][1])
            total["bytes"] += 6 * nnz + 12 * bm["n_protons"] + 8 * nvox
            total["flops"] += 20 * nnz
        return total
    nvox = case["nx"] * case["ny"] * case["nz"]
    if kind == "phantom":
        return {"bytes": 4 * nvox, "flops": 40 * nvox}
    nnz, vb = _size(case), 2 if case["dtype"] == "f16" else 4
    if kind == "sap":
        per = nnz * (4 + vb) + case["rows"] * 16 + 8 * nvox
        return {"bytes": case["iterations"] * per, "flops": case["iterations"] * 4 * nnz}
    if kind == "wepl":
        return {"bytes": 4 * case["rows"] + 4 * nvox, "flops": 20 * nnz}
    return {"bytes": nnz * (4 + vb) + 12 * case["rows"] + (8 if kind == "simulate" else 4) * nvox, "flops": 20 * nnz}


# ------------------------------------------------------ the same results in binary64
MASK32 = 0xFFFFFFFF


def _mul(m, c):
    """High and low words of the 64-bit product of two 32-bit words held in int64."""
    low, high = m * (c & 0xFFFF), m * (c >> 16)
    return (high + (low >> 16)) >> 16, (m * c) & MASK32


def _uniforms(seed, stream, g, draw_no):
    """Two uniforms of [0, 1) per proton from Philox4x32-10, counter (draw, stream, g)."""
    c = [torch.full_like(g, draw_no), torch.full_like(g, stream), g & MASK32, g >> 32]
    k0, k1 = seed & MASK32, (seed >> 32) & MASK32
    for _ in range(10):
        ah, al = _mul(0xD2511F53, c[0])
        bh, bl = _mul(0xCD9E8D57, c[2])
        c = [bh ^ c[1] ^ k0, bl, ah ^ c[3] ^ k1, al]
        k0, k1 = (k0 + 0x9E3779B9) & MASK32, (k1 + 0xBB67AE85) & MASK32
    return [((c[i + 1] << 21) | (c[i] >> 11)).double() * 2.0 ** -53 for i in (0, 2)]


def _normals(seed, stream, g):
    """A pair of standard normals per proton by the polar method, attempt a from draw a."""
    z = torch.zeros(2, g.numel(), dtype=torch.float64, device=g.device)
    todo = torch.arange(g.numel(), device=g.device)
    for a in range(64):
        u = _uniforms(seed, stream, g[todo], a)
        v1, v2 = 2 * u[0] - 1, 2 * u[1] - 1
        s = v1 * v1 + v2 * v2
        ok = (s > 0) & (s < 1)
        f = torch.sqrt(-2 * torch.log(s[ok]) / s[ok])
        z[0, todo[ok]], z[1, todo[ok]] = v1[ok] * f, v2[ok] * f
        todo = todo[~ok]
        if todo.numel() == 0:
            break
    return z[0], z[1]


def _inside(r, p):
    """Whether points p (x, y, z: broadcastable) lie in region r."""
    d = [p[i] - r["center"][i] for i in range(len(p)) if i < len(r["center"])]
    a = math.radians(r["angle_deg"])
    c, s = math.cos(a), math.sin(a)
    u = [c * d[0] + s * d[1], c * d[1] - s * d[0]] + d[2:]
    axes = 3 if r["shape"] == "ellipsoid" and len(p) == 3 else 2
    # (divided by tensors: torch multiplies by the reciprocal of a number)
    semi = [torch.full((1,), v, dtype=torch.float64, device=DEV) for v in r["semi"]]
    return sum((u[i] / semi[i]) ** 2 for i in range(axes)) <= 1.0


def _true_x(ph):
    """The phantom's pixel values, FP64 (flat, x fastest)."""
    dim, n, h = ph["dim"], ph["n"][: ph["dim"]], ph["h"][: ph["dim"]]
    if ph["voxelize"] == "corner_avg":
        offs = [0.0, 1.0]
    elif ph["voxelize"] == "center":
        offs = [0.5]
    else:
        offs = [(i + 0.5) / ph["area_samples"] for i in range(ph["area_samples"])]
    total = torch.zeros(tuple(reversed(n)), dtype=torch.float64, device=DEV)
    shapes = [(1, -1), (-1, 1)] if dim == 2 else [(1, 1, -1), (1, -1, 1), (-1, 1, 1)]
    grids = [[(-n[d] * h[d] / 2 + (torch.arange(n[d], device=DEV, dtype=torch.float64) + o) * h[d]).reshape(shapes[d])
              for o in offs] for d in range(dim)]
    for pz in grids[2] if dim == 3 else [None]:
        for py in grids[1]:
            for px in grids[0]:
                p = [px, py] + ([pz] if dim == 3 else [])
                v = torch.zeros_like(total)
                for r in ph["regions"]:
                    v = torch.where(_inside(r, p), float(np.float32(r["rsp"])), v)
                total += v
    return (total / len(offs) ** dim).reshape(-1)


def _boundary(ph, q, d):
    """Entry and exit parameters of lines q + l d against region 0, and whether they meet."""
    r = ph["regions"][0]
    axes = 3 if r["shape"] == "ellipsoid" and ph["dim"] == 3 else 2
    a = math.radians(r["angle_deg"])
    co, si = math.cos(a), math.sin(a)

    def turn(p, centre):
        p = [p[i] - (r["center"][i] if centre and i < len(r["center"]) else 0.0) for i in range(len(p))]
        return [co * p[0] + si * p[1], co * p[1] - si * p[0]] + p[2:]
    q, d = turn(q, True), turn(d, False)
    w = [1.0 / r["semi"][i] ** 2 for i in range(axes)]
    A = sum(w[i] * d[i] * d[i] for i in range(axes))
    B = sum(w[i] * d[i] * q[i] for i in range(axes))
    C = sum(w[i] * q[i] * q[i] for i in range(axes)) - 1.0
    disc = B * B - A * C
    hit = disc > 0
    t = torch.where(B >= 0, -(B + torch.sqrt(disc.clamp(min=0))), torch.sqrt(disc.clamp(min=0)) - B)
    r1, r2 = t / A, C / t
    return torch.minimum(r1, r2), torch.maximum(r1, r2), hit


def _unit(v):
    n = torch.sqrt(sum(x * x for x in v))
    return [x / n for x in v]


def _paths(ph, bm, g):
    """Every row's path: its straight lines (start, direction, parameter range) before and
    after the curve, and the curve's cubic coefficients and number of chords (0: none)."""
    dim = ph["dim"]
    k = ((g + 1) * bm["n_angles"] - 1) // bm["n_protons"]
    phi = bm["angle0_deg"] + k.double() * bm["dangle_deg"]
    quarter = phi / 90.0
    exact = torch.floor(quarter) == quarter
    m = quarter - 4 * torch.floor(quarter / 4)
    rad = phi * (math.pi / 180.0)
    c = torch.where(exact, (m == 0).double() - (m == 2).double(), torch.cos(rad))
    s = torch.where(exact, (m == 1).double() - (m == 3).double(), torch.sin(rad))
    u0, u1 = _uniforms(bm["seed"], 0, g, 0)
    t = bm["t_range"][0] + (bm["t_range"][1] - bm["t_range"][0]) * u0
    v = bm["v_range"][0] + (bm["v_range"][1] - bm["v_range"][0]) * u1 if dim == 3 else torch.zeros_like(t)
    zero = torch.zeros_like(t)
    q, u, th = [-t * s, t * c, v], [c, s, zero], [-s, c, zero]
    inf = torch.full_like(t, math.inf)
    if bm["path"] == "straight":
        return dict(first=(q, u, -inf, inf), n=torch.zeros_like(g))
    zt, zv = _normals(bm["seed"], 1, g)
    tvi = torch.tan(bm["sigma_in"] * zv) if dim == 3 else zero
    tti = torch.tan(bm["sigma_in"] * zt)
    d0 = _unit([u[i] + tti * th[i] + (tvi if i == 2 else 0.0) for i in range(3)])
    l1, l2, hit = _boundary(ph, q, d0)
    p0 = [q[i] + l1 * d0[i] for i in range(3)]
    p1 = [q[i] + l2 * d0[i] for i in range(3)]
    z1, z2 = _normals(bm["seed"], 2, g)
    z3, z4 = _normals(bm["seed"], 3, g) if dim == 3 else (zero, zero)
    lat, out, rho = bm["sigma_lat"], bm["sigma_out"], bm["rho"]
    if bm["scatter"] == "highland":
        mass = 938.27208816
        energy, pc = bm["energy_mev"] + mass, math.sqrt(bm["energy_mev"] * (bm["energy_mev"] + 2 * mass))
        beta = pc / energy
        x = torch.where(hit, l2 - l1, 1.0)
        w = x / bm["x0_mm"]
        bracket = 1 + 0.038 * (torch.log(w) - math.log(beta * beta))
        out = torch.where(bracket > 0, 13.6 / (beta * pc) * torch.sqrt(w) * bracket, zero)
        lat, rho = out * x / math.sqrt(3.0), math.sqrt(3.0) / 2
    crho = math.sqrt(1 - rho * rho)
    lat_t, ang_t = lat * z1, out * (rho * z1 + crho * z2)
    lat_v, ang_v = lat * z3, out * (rho * z3 + crho * z4)
    td = th[0] * d0[0] + th[1] * d0[1]
    nt = _unit([th[i] - td * d0[i] for i in range(3)])
    nv = _unit([(1.0 if i == 2 else 0.0) - d0[2] * d0[i] for i in range(3)]) if dim == 3 else [zero] * 3
    qd = [q[i] + lat_t * nt[i] + lat_v * nv[i] for i in range(3)]
    _, m2, hit2 = _boundary(ph, qd, d0)
    p1 = [torch.where(hit2, qd[i] + m2 * d0[i], p1[i]) for i in range(3)]
    d1 = _unit([d0[i] + torch.tan(ang_t) * nt[i] + torch.tan(ang_v) * nv[i] for i in range(3)])
    dp = [p1[i] - p0[i] for i in range(3)]
    L = torch.sqrt(sum(x * x for x in dp))
    n = torch.where(hit, torch.ceil(L / bm["step"]).clamp(min=1), zero).nan_to_num(0.0).long()
    c1 = [L * d0[i] for i in range(3)]
    c2 = [3 * dp[i] - 2 * L * d0[i] - L * d1[i] for i in range(3)]
    c3 = [-2 * dp[i] + L * d0[i] + L * d1[i] for i in range(3)]
    start = [torch.where(hit, p0[i], q[i]) for i in range(3)]
    return dict(first=(start, d0, -inf, torch.where(hit, 0.0, inf)), curve=(p0, c1, c2, c3), end=p1,
                last=(p1, d1, zero, inf), n=n)


def _lines(ph, line, use):
    """Lines clipped to the grid box: start point, end point, whether they meet it."""
    (a, d, lo, hi), dim = line, ph["dim"]
    ok = use.clone()
    for i in range(dim):
        m = ph["n"][i] * ph["h"][i] / 2
        flat = d[i] == 0
        di = torch.where(flat, 1.0, d[i])
        t1, t2 = (-m - a[i]) / di, (m - a[i]) / di
        ok &= ~(flat & ((a[i] < -m) | (a[i] > m)))
        lo = torch.where(flat, lo, torch.maximum(lo, torch.minimum(t1, t2)))
        hi = torch.where(flat, hi, torch.minimum(hi, torch.maximum(t1, t2)))
    ok &= lo < hi
    lo, hi = torch.where(ok, lo, 0.0), torch.where(ok, hi, 0.0)
    return [a[i] + lo * d[i] for i in range(dim)], [a[i] + hi * d[i] for i in range(dim)], ok


def _trace_rows(ph, bm, g):
    """Entries per row, columns and lengths (FP64) of rows g."""
    dim, R = ph["dim"], g.numel()
    p = _paths(ph, bm, g)
    curved = p["n"] > 0
    s0, e0, ok0 = _lines(ph, p["first"], torch.ones(R, dtype=torch.bool, device=DEV))
    # segments of every row, in order: (rows, segments) tensors of their two ends per axis
    A, E, use = [x[:, None] for x in s0], [x[:, None] for x in e0], ok0[:, None]
    if "curve" in p:
        top = int(p["n"].max())
        j = torch.arange(top + 1, device=DEV)
        sj = j[None, :].double() / p["n"].clamp(min=1)[:, None].double()
        pts = []
        for i in range(dim):
            k0, k1, k2, k3 = (x[i][:, None] for x in p["curve"])
            v = ((k3 * sj + k2) * sj + k1) * sj + k0
            pts.append(torch.where(j[None, :] == p["n"][:, None], p["end"][i][:, None], v))
        s2, e2, ok2 = _lines(ph, p["last"], curved)
        on = (j[None, :-1] < p["n"][:, None]) & curved[:, None]
        ca, ce = [v[:, :-1] for v in pts], [v[:, 1:] for v in pts]
        inside = on & True
        for i in range(dim):
            m = ph["n"][i] * ph["h"][i] / 2
            inside &= (ca[i].abs() <= m) & (ce[i].abs() <= m)
        if bool((on & ~inside).any()):   # chords that leave the box are clipped to it
            chord = (ca, [ce[i] - ca[i] for i in range(dim)], torch.zeros_like(ca[0]), torch.ones_like(ca[0]))
            cs, cl, ok = _lines(ph, chord, on)
            ca = [torch.where(inside, ca[i], cs[i]) for i in range(dim)]
            ce = [torch.where(inside, ce[i], cl[i]) for i in range(dim)]
            on = on & (inside | ok)
        A = [torch.cat([A[i], torch.where(on, ca[i], 0.0), s2[i][:, None]], 1) for i in range(dim)]
        E = [torch.cat([E[i], torch.where(on, ce[i], 0.0), e2[i][:, None]], 1) for i in range(dim)]
        use = torch.cat([use, on, ok2[:, None]], 1)
    seg = torch.sqrt(sum((E[i] - A[i]) ** 2 for i in range(dim))) * use
    arc = torch.cumsum(seg, 1)
    before = (arc - seg).reshape(-1)
    S = use.shape[1]
    rows, where, steps = [], [], []
    stride, first = 1, torch.zeros(R, dtype=torch.int64, device=DEV)
    lead = use.double().argmax(1)
    for i in range(dim):
        o, h, n = -ph["n"][i] * ph["h"][i] / 2, ph["h"][i], ph["n"][i]
        ia = torch.floor((A[i] - o) / h).clamp(0, n - 1).long()
        ie = torch.floor((E[i] - o) / h).clamp(0, n - 1).long()
        first += stride * ia.gather(1, lead[:, None])[:, 0]
        count = ((ie - ia).abs() * use).reshape(-1)
        some = torch.nonzero(count)[:, 0]
        c = count[some]
        which = torch.repeat_interleave(some, c)
        step = torch.arange(which.numel(), device=DEV) - torch.repeat_interleave(torch.cumsum(c, 0) - c, c)
        ai, ei, av, ev = (x.reshape(-1)[which] for x in (ia, ie, A[i], E[i]))
        up = ei > ai
        plane = o + (ai + torch.where(up, 1 + step, -step)).double() * h
        lam = ((plane - av) / (ev - av)).clamp(0, 1)
        rows.append(which // S)
        where.append(before[which] + lam * seg.reshape(-1)[which])
        steps.append(torch.where(up, stride, -stride))
        stride *= n
    hit = torch.nonzero(use.any(1))[:, 0]
    rows.append(hit)
    where.append(arc[hit, -1])
    steps.append(torch.zeros_like(hit))
    rows, where, steps = torch.cat(rows), torch.cat(where), torch.cat(steps)
    at = torch.sort(where, stable=True).indices
    at = at[torch.sort(rows[at], stable=True).indices]
    rows, where, steps = rows[at], where[at], steps[at]
    counts = torch.bincount(rows, minlength=R)
    begin = torch.cumsum(counts, 0) - counts
    head = torch.arange(rows.numel(), device=DEV) == begin[rows]
    prev = torch.where(head, 0.0, torch.roll(where, 1))
    moved = torch.cumsum(steps, 0) - steps
    cols = first[rows] + moved - moved[begin[rows]]
    return counts, cols, where - prev


def _trace(c, seed, dtype=None):
    """The system (row_ptr, cols, vals, b, x) of a case in FP64, or with values and b
    rounded as a program has them in hand (dtype)."""
    cfg = prepare(c, seed)["cfg"] if c["kind"] == "simulate" else _config(c, seed)
    ph, bm = cfg["phantom"], cfg["beam"]
    x = _true_x(ph).float().double()   # b is taken with the stored FP32 x
    rows = c["rows"]
    out = dict(counts=[], cols=[], vals=[], b=[])
    chunk = 8192 if c["path"] == "hermite" else 65536
    for r in range(0, rows, chunk):
        g = torch.arange(r, min(rows, r + chunk), device=DEV)
        counts, cols, vals = _trace_rows(ph, bm, g)
        at = torch.repeat_interleave(torch.arange(g.numel(), device=DEV), counts)
        b = torch.zeros(g.numel(), dtype=torch.float64, device=DEV).index_add_(0, at, vals * x[cols])
        if bm["noise_rel"] > 0:
            b = b * (1 + bm["noise_rel"] * _normals(bm["seed"], 4, g)[0])
        if dtype:
            vals, b = vals.half() if dtype == "f16" else vals.float(), b.float()
        for key, v in zip(("counts", "cols", "vals", "b"), (counts, cols.int(), vals, b)):
            out[key].append(v)
    row_ptr = torch.zeros(rows + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.cumsum(torch.cat(out["counts"]), 0)
    return row_ptr, torch.cat(out["cols"]), torch.cat(out["vals"]), torch.cat(out["b"]), x


def _reconstruct(c, seed):
    """String-averaging projections in FP64, all strings side by side."""
    row_ptr, cols, vals, b, _ = _trace(c, seed, c["dtype"])
    m, n, M = c["rows"], c["nx"] * c["ny"], c["strings"]
    t = torch.arange(M, device=DEV)
    s0, s1 = t * m // M, (t + 1) * m // M
    width = int((row_ptr[1:] - row_ptr[:-1]).max())
    lane = torch.arange(width, device=DEV)[None, :]
    coef = torch.zeros(m, dtype=torch.float64, device=DEV)
    x = torch.zeros(n, dtype=torch.float64, device=DEV)
    relax = float(np.float32(c["relax"]))
    norm = torch.zeros(M, n, dtype=torch.float64, device=DEV)
    for it in range(c["iterations"]):
        y = x[None, :].repeat(M, 1)
        for p in range(int((s1 - s0).max())):
            live = s0 + p < s1
            i = torch.where(live, s0 + p, 0)
            on = live[:, None] & (lane < (row_ptr[i + 1] - row_ptr[i])[:, None])
            e = torch.where(on, row_ptr[i][:, None] + lane, 0)
            col, v = cols[e].long(), torch.where(on, vals[e].double(), 0.0)
            if it == 0:
                # the norm of the row as a vector: entries that share a column add up
                norm.scatter_add_(1, col, v)
                sq = (v * norm.gather(1, col)).sum(1)
                norm.scatter_(1, col, 0.0)
                coef[i] = torch.where(live, torch.where(sq > 0, relax / sq, 0.0), coef[i])
            a = torch.where(live, (b[i].double() - (v * y.gather(1, col)).sum(1)) * coef[i], 0.0)
            y.scatter_add_(1, col, a[:, None] * v)
        x = y.mean(0)
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return None
    if kind == "phantom":
        return {"x": _true_x(prepare(case, seed)["phantom"])}
    if kind == "sap":
        return {"x": _reconstruct(case, seed)}
    if _size(case) > (3.0e8 if case["path"] == "straight" else 2.5e8):
        return None
    _, _, vals, b, x = _trace(case, seed)
    if kind == "wepl":
        return {"b": b}
    if case["chord"] > 0 and kind == "emit":
        vals = torch.full_like(vals, case["chord"])
    if kind == "simulate":
        return dict(row_ptr=None, cols=None, vals=vals, b=b, x=x, nnz=None)
    whole = torch.zeros(_capacity(_phantom(case), _make_beam(case, seed)), dtype=torch.float64, device=DEV)
    whole[: vals.numel()] = vals
    return {"jobs": [dict(row_ptr=None, cols=None, vals=whole, b=b, x=x)], "nnz": None}
