"""Performance cases: the tracking calls that users of this library make.

A case is a dict of plain values.  `prepare` builds what a program holds before the call (flow
fields loaded on the GPU, released particles, output buffers), `run` makes one pass through the
public entry points of `paper_2302_13590_amd.pt`, `exact` follows the same particles in plain
64-bit torch arithmetic, and `work` counts the bytes and operations a pass cannot do without.

The shapes are those of the repository's own workloads (C1 - C7 and the first test case's
two-dimensional aquifer): lognormal conductivity with an exponential covariance, heads fixed on
the west and east faces, optional recharge and pumping wells, a flow solve, and particles released
near the inlet or over the whole domain.

Keys of a case:
  kind       "field" (one steady field), "groups" (several realisations in one call), "transient"
             (one field per time step) or "quadtree"
  nx, ny, nz, dx, dz, sigma2, corr   grid, cell sizes, variance and correlation length of ln K
  n          particles (all groups together)
  release    "inlet" (the first tenth of the columns), "column" (the first column), "line" (a line
             across the inlet) or "domain"
  wells      pumping-well columns (sink cells); recharge: m/d through the top
  precision  "fp64" or "mixed"; direction: 1 or -1; t_max: limit in days, 0 for none
  snaps      snapshot times (timeseries) or 0; pathlines: whether the pathline records are wanted
  entry      "track" (pt.track with its defaults), "tuned" (pt.track with the launch that the
             autotuner records), "noalloc" (pt_track_noalloc) or "realisation" (load the field from
             host arrays, track, release it)
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

from paper_2302_13590_amd import pt

FNV_OFFSET = 0xCBF29CE484222325
POROSITY = 0.3
HUGE_T = math.inf
# a transient run: the pumping rate of each time step and the step ends (days)
RATES = (0.0, 250.0, 500.0, 750.0, 1000.0, 1000.0, 750.0, 500.0, 250.0, 0.0, 0.0, 0.0)
ENDS = (50.0, 100.0, 150.0, 200.0, 300.0, 400.0, 600.0, 800.0, 1200.0, 1600.0, 2400.0, math.inf)


def _case(kind="field", nx=100, ny=100, nz=10, dx=10.0, dz=2.0, sigma2=1.0, corr=5.0, n=100_000, release="inlet",
          wells=0, recharge=0.0, precision="fp64", direction=1, t_max=0.0, snaps=0, pathlines=False, entry="track",
          fields=1, name=None):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, dx=dx, dz=dz, sigma2=sigma2, corr=corr, n=n, release=release, wells=wells,
             recharge=recharge, precision=precision, direction=direction, t_max=t_max, snaps=snaps, pathlines=pathlines,
             entry=entry, fields=fields)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # a first look at a small homogeneous model: one short call, latency and launches count
        _case(name="small_homogeneous", nx=40, ny=40, nz=1, dz=10.0, sigma2=0.0, n=1000, release="column"),
        # a serving loop that must not allocate: backward travel of a few thousand points of
        # interest over ten years (their capture zones), many calls in a row
        _case(name="noalloc_capture", n=4096, release="domain", wells=1, direction=-1, t_max=3650.0, entry="noalloc"),
        # the two-dimensional aquifer of the scheduling study: few particles, very long paths
        _case(name="line_2d", nx=1500, ny=300, nz=1, dx=1.0, dz=1.0, sigma2=2.5, corr=10.0, n=10_000, release="line"),
        # one realisation of a Monte-Carlo loop: the flow model hands over host arrays, a moderate
        # release is tracked, the field is let go
        _case(name="realisation", n=100_000, entry="realisation"),
        # a full release through a mildly heterogeneous field, the launch taken from the tuner
        _case(name="endpoint_fp64", n=1_000_000, entry="tuned"),
        # the same in mixed precision
        _case(name="endpoint_mixed", n=1_000_000, precision="mixed", entry="tuned"),
        # a large strongly heterogeneous field with wells and recharge, particles everywhere
        _case(name="wells_recharge", nx=200, ny=200, nz=20, sigma2=4.0, corr=8.0, n=4_000_000, release="domain", wells=2,
              recharge=1e-4),
        # sixteen realisations and 64 release groups of very different sizes in one call
        _case(name="groups", kind="groups", fields=16, sigma2=2.0, n=6_000_000, entry="tuned"),
        # positions at 100 times, breakthrough and plume snapshots
        _case(name="timeseries", nx=200, ny=200, nz=20, sigma2=2.0, corr=8.0, n=200_000, release="column", snaps=100,
              t_max=1e5),
        # twelve time steps with a well that switches on and off, releases every 20 d, weak sinks
        _case(name="transient", kind="transient", fields=12, n=500_000, wells=1, recharge=1e-4),
        # a layered quadtree grid refined around two wells
        _case(name="quadtree", kind="quadtree", nx=256, ny=256, nz=3, dx=2.5, dz=5.0, corr=12.0, n=300_000,
              release="domain", wells=2, recharge=2e-4),
        # full pathlines of a moderate release: count pass, records
        _case(name="pathlines", n=50_000, pathlines=True),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["small", "line", "field", "field", "groups", "timeseries", "transient", "quadtree", "pathlines"])
    box = dict(nx=rng.randint(37, 160), ny=rng.randint(33, 140), nz=rng.randint(3, 17),
               sigma2=round(rng.uniform(0.3, 2.5), 3), corr=round(rng.uniform(3.0, 9.0), 2))
    prec = rng.choice(["fp64", "fp64", "mixed"])
    if kind == "small":
        entry = rng.choice(["track", "noalloc", "realisation"])
        return _case(nx=rng.randint(21, 80), ny=rng.randint(17, 90), nz=rng.randint(1, 5), sigma2=round(rng.uniform(0.1, 1.0), 3),
                     corr=4.0, n=size(500, 20_000), release=rng.choice(["inlet", "domain"]), entry=entry,
                     direction=rng.choice([1, -1]), t_max=rng.choice([0.0, 2000.0]))
    if kind == "line":
        return _case(nx=rng.randint(301, 1500), ny=rng.randint(101, 300), nz=1, dx=1.0, dz=1.0, sigma2=round(rng.uniform(0.1, 4.0), 3),
                     corr=10.0, n=size(1000, 300_000), release="line")
    if kind == "groups":
        return _case(kind="groups", fields=rng.randint(2, 12), n=size(50_000, 3_000_000), precision=prec,
                     entry=rng.choice(["track", "tuned"]), **dict(box, sigma2=1.0 if prec == "mixed" else 2.0))
    if kind == "timeseries":
        return _case(n=size(5_000, 200_000), release="column", snaps=rng.randint(5, 120), t_max=1e5, precision=prec,
                     **dict(box, sigma2=1.0) if prec == "mixed" else box)
    if kind == "transient":
        return _case(kind="transient", fields=12, n=size(5_000, 500_000), wells=1, recharge=1e-4,
                     nx=box["nx"], ny=box["ny"], nz=box["nz"])
    if kind == "quadtree":
        return _case(kind="quadtree", nx=4 * rng.randint(24, 64), ny=4 * rng.randint(24, 64), nz=3, dx=2.5, dz=5.0, corr=12.0,
                     n=size(5_000, 400_000), release="domain", wells=2, recharge=2e-4)
    if kind == "pathlines":
        return _case(n=size(2_000, 50_000), pathlines=True, direction=rng.choice([1, -1]), release=rng.choice(["inlet", "domain"]), **box)
    return _case(n=size(20_000, 2_000_000), release=rng.choice(["inlet", "domain"]), wells=rng.choice([0, 1, 2]), recharge=1e-4,
                 entry=rng.choice(["track", "tuned"]), precision=prec, direction=rng.choice([1, -1]), t_max=rng.choice([0.0, 5000.0]),
                 **dict(box, sigma2=1.0) if prec == "mixed" else box)


# ------------------------------------------------------------------------------------------- fields

def _gaussian(shape, corr, gen):
    """Standardised Gaussian field with covariance exp(-|h|/corr), by circulant embedding."""
    lag = []
    for n in shape:
        m = 1 if n == 1 else max(2 * n, n + math.ceil(4 * corr))
        a = torch.arange(m + (m > 1 and m % 2), dtype=torch.float64, device="cuda")
        lag.append(torch.minimum(a, len(a) - a))
    h = torch.sqrt(lag[0][:, None, None] ** 2 + lag[1][None, :, None] ** 2 + lag[2][None, None, :] ** 2)
    eig = torch.fft.rfftn(torch.exp(-h / corr)).real.clamp_(min=0.0)
    z = torch.randn(h.shape, dtype=torch.float64, device="cuda", generator=gen)
    y = torch.fft.irfftn(torch.sqrt(eig) * torch.fft.rfftn(z), s=h.shape)[:shape[0], :shape[1], :shape[2]]
    y = y - y.mean()
    return y / y.std()


def _flows(K, dx, dz, h_west, h_east, recharge, source):
    """Face flows of B fields: harmonic conductances, heads fixed on the west and east faces, conjugate
    gradients with a diagonal preconditioner.  K, source: [B, nz, ny, nx]."""
    area_x, area_z = dx * dz, dx * dx
    b, nz, ny, nx = K.shape
    cx = K.new_zeros(b, nz, ny, nx + 1)
    cy = K.new_zeros(b, nz, ny + 1, nx)
    cz = K.new_zeros(b, nz + 1, ny, nx)
    cx[..., 1:-1] = 2 * area_x / dx / (1 / K[..., 1:] + 1 / K[..., :-1])
    cx[..., 0], cx[..., -1] = 2 * area_x / dx * K[..., 0], 2 * area_x / dx * K[..., -1]
    cy[..., 1:-1, :] = 2 * area_x / dx / (1 / K[..., 1:, :] + 1 / K[..., :-1, :])
    cz[:, 1:-1] = 2 * area_z / dz / (1 / K[:, 1:] + 1 / K[:, :-1])
    diag = cx[..., 1:] + cx[..., :-1] + cy[..., 1:, :] + cy[..., :-1, :] + cz[:, 1:] + cz[:, :-1]
    ix, iy, iz = cx[..., 1:-1].contiguous(), cy[..., 1:-1, :].contiguous(), cz[:, 1:-1].contiguous()

    def apply(p):
        q = diag * p
        q[..., 1:] -= ix * p[..., :-1]
        q[..., :-1] -= ix * p[..., 1:]
        q[..., 1:, :] -= iy * p[..., :-1, :]
        q[..., :-1, :] -= iy * p[..., 1:, :]
        if nz > 1:
            q[:, 1:] -= iz * p[:, :-1]
            q[:, :-1] -= iz * p[:, 1:]
        return q

    def dot(u, v):
        return (u * v).sum((1, 2, 3), keepdim=True)

    rhs = source.clone()
    rhs[:, -1] += recharge * area_z
    rhs[..., 0] += cx[..., 0] * h_west
    rhs[..., -1] += cx[..., -1] * h_east
    x = torch.linspace(h_west, h_east, nx, dtype=K.dtype, device=K.device).expand_as(K).contiguous()
    r = rhs - apply(x)
    z = r / diag
    p, rz, target = z, dot(r, z), 1e-22 * dot(rhs, rhs)
    for it in range(20000):
        q = apply(p)
        alpha = rz / dot(p, q)
        x = x + alpha * p
        r = r - alpha * q
        if it % 100 == 99 and bool((dot(r, r) <= target).all()):
            break
        z = r / diag
        new = dot(r, z)
        p = z + (new / rz) * p
        rz = new
    qx, qy, qz = torch.zeros_like(cx), torch.zeros_like(cy), torch.zeros_like(cz)
    qx[..., 1:-1] = ix * (x[..., :-1] - x[..., 1:])
    qx[..., 0] = cx[..., 0] * (h_west - x[..., 0])
    qx[..., -1] = cx[..., -1] * (x[..., -1] - h_east)
    qy[..., 1:-1, :] = iy * (x[..., :-1, :] - x[..., 1:, :])
    qz[:, 1:-1] = iz * (x[:, :-1] - x[:, 1:])
    qz[:, -1] = -recharge * area_z
    return qx, qy, qz


def _grids(case, gen):
    """The case's structured fields as descriptions that pt.pt_load_grid takes (device tensors)."""
    shape = (case["nz"], case["ny"], case["nx"])
    f = case["fields"]
    spread = torch.linspace(0.25, 1.75, f).tolist() if case["kind"] == "groups" else [1.0] * f
    fields = []
    for b in range(f):
        if case["kind"] == "transient" and b:
            fields.append(fields[0])
            continue
        y = _gaussian(shape, case["corr"], gen) if case["sigma2"] > 0 else torch.zeros(shape, dtype=torch.float64, device="cuda")
        fields.append(10.0 * torch.exp(math.sqrt(case["sigma2"] * spread[b]) * y))
    K = torch.stack(fields)
    if case["kind"] == "quadtree":      # aquifer, aquitard, aquifer
        K[:, 0] *= 2.0
        K[:, 1] *= 0.005
    source = torch.zeros_like(K)
    flags = torch.ones(K.shape, dtype=torch.int32, device="cuda")
    for w in range(case["wells"]):
        i, j = case["nx"] * (w + 1) // (case["wells"] + 1), case["ny"] // 2 + w
        if case["kind"] == "quadtree":  # one well in the top and one in the bottom aquifer
            layers = [0 if w == 0 else case["nz"] - 1]
        else:
            layers = range(case["nz"])
        for b in range(f):
            rate = RATES[b] if case["kind"] == "transient" else 300.0
            if rate > 0:
                for k in layers:
                    source[b, k, j, i] = -rate / len(layers)
                    flags[b, k, j, i] = 3
    heads = (1510.0, 10.0) if case["nz"] == 1 and case["dx"] == 1.0 else (10.0, 0.0)
    qx, qy, qz = _flows(K, case["dx"], case["dz"], heads[0], heads[1], case["recharge"], source)
    return [types.SimpleNamespace(nx=case["nx"], ny=case["ny"], nz=case["nz"], dx=case["dx"], dy=case["dx"], dz=case["dz"],
                                  x0=0.0, y0=0.0, z0=0.0, qx=qx[b], qy=qy[b], qz=qz[b], porosity=None,
                                  porosity_scalar=POROSITY, flags=flags[b]) for b in range(f)]


def _quadtree(case, g):
    """Merge the fine grid's columns far from the wells into blocks of 2 x 2 and 4 x 4 cells; a
    merged face keeps one subface per neighbour, with the summed fine flows."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    fine = {k: getattr(g, k).cpu().numpy() for k in ("qx", "qy", "qz", "flags")}
    wells = np.argwhere(fine["flags"].max(0) & 2)[:, ::-1]

    def far(step, r):
        jj, ii = np.meshgrid(np.arange(0, ny, step) + step / 2, np.arange(0, nx, step) + step / 2, indexing="ij")
        d = np.min(np.hypot(ii[..., None] - wells[:, 0], jj[..., None] - wells[:, 1]), axis=-1)
        return np.kron(d > r, np.ones((step, step), bool))

    size = np.where(far(4, 28.0), 4, np.where(far(2, 10.0), 2, 1))
    jj, ii = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
    head = (jj % size == 0) & (ii % size == 0)
    index = np.cumsum(head).reshape(ny, nx) - 1
    owner2 = index[jj - jj % size, ii - ii % size]
    per, (cj, ci) = int(head.sum()), np.nonzero(head)
    cs = size[head]
    owner = owner2[None] + per * np.arange(nz)[:, None, None]
    ncell = per * nz
    kk = np.repeat(np.arange(nz), per)
    i0, j0, s = np.tile(ci, nz), np.tile(cj, nz), np.tile(cs, nz)
    box = np.stack([i0 * g.dx, j0 * g.dy, kk * g.dz, s * g.dx, s * g.dy, np.full(ncell, g.dz)], axis=1).astype(np.float64)
    cell, face, pos, nb, q = [], [], [], [], []

    def add(mask, f, t, neighbour, flow):   # fine faces [nz, ny, nx] on a block's face f
        m = np.broadcast_to(mask, owner.shape)
        cell.append(owner[m])
        face.append(np.full(int(m.sum()), f))
        pos.append(np.broadcast_to(t, owner.shape)[m])
        nb.append(neighbour[m])
        q.append(flow[m])

    pad = np.pad(owner, 1, constant_values=-1)
    jr, ir = jj % size, ii % size
    add(ir == 0, 0, jr, pad[1:-1, 1:-1, :-2], fine["qx"][:, :, :-1])
    add(ir == size - 1, 1, jr, pad[1:-1, 1:-1, 2:], fine["qx"][:, :, 1:])
    add(jr == 0, 2, ir, pad[1:-1, :-2, 1:-1], fine["qy"][:, :-1])
    add(jr == size - 1, 3, ir, pad[1:-1, 2:, 1:-1], fine["qy"][:, 1:])
    add(size > 0, 4, jr * size + ir, pad[:-2, 1:-1, 1:-1], fine["qz"][:-1])
    add(size > 0, 5, jr * size + ir, pad[2:, 1:-1, 1:-1], fine["qz"][1:])
    cell, face, pos, nb, q = (np.concatenate(a) for a in (cell, face, pos, nb, q))
    o = np.lexsort((pos, face, cell))
    cell, face, pos, nb, q = cell[o], face[o], pos[o], nb[o], q[o]
    key = cell * 6 + face
    start = np.nonzero(np.r_[True, (key[1:] != key[:-1]) | (nb[1:] != nb[:-1])])[0]
    last = np.r_[start[1:], len(key)] - 1
    lo, hi = np.zeros((len(start), 2)), np.ones((len(start), 2))
    flat = face[start] < 4
    lo[flat, 0] = pos[start][flat] / s[cell[start]][flat]
    hi[flat, 0] = (pos[last][flat] + 1) / s[cell[start]][flat]
    off = np.zeros(6 * ncell + 1, np.int64)
    np.add.at(off, key[start] + 1, 1)
    flags = np.zeros(ncell, np.int32)
    np.bitwise_or.at(flags, owner.ravel(), fine["flags"].ravel())
    return types.SimpleNamespace(ncell=ncell, box=box, sub_off=np.cumsum(off).astype(np.int32), sub_nb=nb[start].astype(np.int32),
                                 sub_q=np.add.reduceat(q, start), sub_lo=lo, sub_hi=hi, flags=flags, porosity=None,
                                 porosity_scalar=POROSITY, owner=torch.from_numpy(owner).cuda(), i0=torch.from_numpy(i0).cuda(),
                                 j0=torch.from_numpy(j0).cuda(), s=torch.from_numpy(s).cuda())


# ------------------------------------------------------------------------------------------- particles

_FIELDS = (("xi", 8), ("eta", 8), ("zeta", 8), ("t", 8), ("path_hash", 8), ("cell", 4), ("status", 4), ("ncross", 4))
_DTYPES = dict(path_hash=torch.int64, cell=torch.int32, status=torch.int32, ncross=torch.int32)


def _views(arena, n):
    """The particle arrays as views of one allocation (each 512-byte aligned)."""
    out, at = {}, 0
    for name, width in _FIELDS:
        out[name] = arena[at:at + n * width].view(_DTYPES.get(name, torch.float64))
        at += (n * width + 511) // 512 * 512
    return pt.DeviceParticles(**out)


def _released(case, gen, quad):
    n, nx, ny, nz = case["n"], case["nx"], case["ny"], case["nz"]
    arena = torch.zeros(sum((n * w + 511) // 512 * 512 for _, w in _FIELDS), dtype=torch.uint8, device="cuda")
    p = _views(arena, n)

    def integers(hi):
        return torch.randint(0, hi, (n,), device="cuda", generator=gen)

    def uniform():
        return torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)

    wide = {"inlet": max(1, nx // 10), "column": 1, "line": 1, "domain": nx}[case["release"]]
    i, j, k = integers(wide), integers(ny), integers(nz)
    p.xi.copy_(uniform())
    p.eta.copy_(uniform())
    p.zeta.copy_(uniform())
    if case["release"] == "line":
        i = i + min(10, nx - 1)
        p.xi.zero_()
        p.zeta.fill_(0.5)
    if quad is not None:
        k = torch.zeros_like(k)
        c = quad.owner[k, j, i]
        p.xi.copy_((i - quad.i0[c] + p.xi) / quad.s[c])
        p.eta.copy_((j - quad.j0[c] + p.eta) / quad.s[c])
        p.cell.copy_(c)
    else:
        p.cell.copy_((k * ny + j) * nx + i)
    if case["kind"] == "transient":
        p.t.copy_(20.0 * (torch.arange(n, device="cuda") % 10))
    p.path_hash.fill_(FNV_OFFSET - (1 << 64))
    return arena, p


def _groups(case):
    """64 release groups, sizes log-uniform over three decades, dealt to the realisations in turn."""
    rng = np.random.Generator(np.random.PCG64(case["n"]))
    w = np.exp(rng.uniform(math.log(1e3), math.log(2e6), size=64))
    offs = np.r_[0, np.floor(np.cumsum(w) / w.sum() * case["n"])].astype(np.int64)
    offs[-1] = case["n"]
    return offs, (np.arange(64) % case["fields"]).astype(np.int32)


class State:
    """What a program holds between calls; its grids are released with it."""

    def __del__(self):
        for g in getattr(self, "grids", []):
            g.release()


def _options(case):
    o = dict(precision=pt.PT_MIXED if case["precision"] == "mixed" else pt.PT_FP64, direction=case["direction"])
    if case["t_max"] > 0:
        o["t_max"] = case["t_max"]
    if case["kind"] == "transient":
        o.update(tstep_end=np.array(ENDS), stop_at_sink=0)
    if case["snaps"]:
        o.update(mode=pt.PT_TIMESERIES, snap_times=_snap_times(case))
    if case["entry"] == "tuned":
        o.update(schedule=pt.PT_SCHED_STATIC, sort=pt.PT_SORT_CELL, layout=pt.PT_LAYOUT_CELL, use_graph=1,
                 block=256 if case["precision"] == "mixed" else 64)
    return o


def _snap_times(case):
    return 10.0 ** (5.0 * np.arange(case["snaps"]) / max(1, case["snaps"] - 1))


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    descs = _grids(case, gen)
    quad = _quadtree(case, descs[0]) if case["kind"] == "quadtree" else None
    arena, parts = _released(case, gen, quad)
    return descs, quad, arena, parts


def prepare(case, seed):
    descs, quad, pristine, _ = _inputs(case, seed)
    s = State()
    s.case, s.n, s.pristine = case, case["n"], pristine
    s.arena = pristine.clone()
    s.parts = _views(s.arena, s.n)
    s.options = _options(case)
    s.options["out_xyz"] = s.out = torch.empty(s.n, 3, dtype=torch.float64, device="cuda")
    s.group = dict(zip(("group_offsets", "group_grid"), _groups(case))) if case["kind"] == "groups" else {}
    s.grids = []
    if case["snaps"]:
        s.options["snap_xyz"] = s.snap = torch.empty(s.n, case["snaps"], 3, dtype=torch.float64, device="cuda")
    if case["pathlines"]:
        # record storage for a run of this size, with room to spare
        s.lines = pt.Pathlines(torch.zeros(s.n + 1, dtype=torch.int64, device="cuda"), pt.path_record_buffer(_capacity(case)).zero_())
        s.options.update(mode=pt.PT_PATHLINE, path_offsets=s.lines.offsets)
    if case["entry"] == "realisation":
        s.host = descs[0]
        for k in ("qx", "qy", "qz", "flags"):
            setattr(s.host, k, getattr(s.host, k).cpu().numpy())
    elif quad is not None:
        s.grids = [pt.pt_load_quad_grid(quad)]
    else:
        s.grids = [pt.pt_load_grid(d) for d in descs]
    if case["entry"] == "noalloc":
        s.counts = torch.zeros(pt.PT_COUNTS_WORDS, dtype=torch.int64, device="cuda")
        s.options = pt.make_opts(**s.options)
    return s


def run(s):
    s.arena.copy_(s.pristine)       # a fresh release
    out = {}
    if s.case["entry"] == "noalloc":
        pt.pt_track_noalloc(s.grids, s.parts, s.options, s.counts)
        out["counts"] = s.counts
    elif s.case["entry"] == "realisation":
        grid = pt.pt_load_grid(s.host)
        summary = pt.track([grid], s.parts, **s.options)
        grid.release()
        out.update(crossings=summary["crossings"])
    elif s.case["pathlines"]:
        lines = s.lines
        pt.track(s.grids, s.parts, path_count_only=1, **s.options)
        summary = pt.track(s.grids, s.parts, path_cap=len(lines.records), path_records=lines.records, **s.options)
        out.update(crossings=summary["crossings"], dropped=summary["path_dropped"], offsets=lines.offsets, record_t=lines.t,
                   record_xyz=lines.xyz, record_cell=lines.cell, record_face=lines.face)
    else:
        summary = pt.track(s.grids, s.parts, **s.group, **s.options)
        out.update(crossings=summary["crossings"], tracked=summary["n_tracked"])
    p = s.parts
    out.update(xi=p.xi, eta=p.eta, zeta=p.zeta, t=p.t, cell=p.cell, status=p.status, ncross=p.ncross, path_hash=p.path_hash,
               xyz=s.out)
    if s.case["snaps"]:
        out["snap_xyz"] = s.snap
    return out


def _mean_path(case):
    """Crossings per particle, roughly: the columns ahead, and the sideways steps on the way."""
    ahead = {"inlet": 0.95, "column": 1.0, "line": 1.0, "domain": 0.5}[case["release"]] * case["nx"]
    side = 0.0 if case["sigma2"] == 0 else (0.35 if case["nz"] == 1 else 0.6)
    if case["t_max"] > 0 and not case["snaps"]:
        ahead *= 0.5
    if case["kind"] == "quadtree":
        ahead *= 0.35
    return ahead * (1.0 + side)


def _capacity(case):
    return int(2.0 * case["n"] * _mean_path(case))


def work(case):
    """Each input once (particle state 52 B, a 64-byte or 32-byte cell record), each output once
    (state, final position, snapshots, records); ~150 64-bit operations for a crossing."""
    n, cells = case["n"], case["nx"] * case["ny"] * case["nz"] * case["fields"]
    crossings = n * _mean_path(case)
    b = n * (52 + 52 + 24) + cells * (32 if case["precision"] == "mixed" else 64) + n * case["snaps"] * 24
    if case["pathlines"]:
        b += int(crossings * 40)
    if case["entry"] == "realisation":
        b += cells * 28
    return {"bytes": int(b), "flops": int(150 * crossings + 60 * n * case["snaps"])}


# ------------------------------------------------------------------------------------------- 64-bit values

def _psi(y):
    return torch.where(y == 0, torch.ones_like(y), torch.expm1(y) / torch.where(y == 0, torch.ones_like(y), y))


def _exit_times(u1, u2, x):
    A = u2 - u1
    up = u1 + A * x
    high = up > 0
    ue = torch.where(high, u2, u1)
    reach = (high & (ue > 0)) | ((up < 0) & (ue < 0))
    e = high.to(x.dtype)
    r = torch.where(reach, (e - x) / torch.where(up == 0, torch.ones_like(up), up), torch.zeros_like(x))
    y = A * r
    slow = y < -0.5
    ratio = torch.where(slow & reach, ue / torch.where(up == 0, torch.ones_like(up), up), torch.ones_like(up))
    dt = torch.where(slow, torch.log(ratio) / torch.where(A == 0, torch.ones_like(A), A),
                     torch.where(y == 0, r, r * torch.log1p(torch.where(slow, torch.zeros_like(y), y)) / torch.where(y == 0, torch.ones_like(y), y)))
    return torch.where(reach, dt.clamp(min=0.0), torch.full_like(dt, HUGE_T)), A, up, e


def _tables(case, descs, quad):
    """Face velocities [fields * cells, 6] (low, high of i, j, k) and flags."""
    if quad is not None:
        off = torch.from_numpy(quad.sub_off).cuda().long()
        total = torch.zeros(6 * quad.ncell, dtype=torch.float64, device="cuda")
        which = torch.repeat_interleave(torch.arange(6 * quad.ncell, device="cuda"), off[1:] - off[:-1])
        total.index_add_(0, which, torch.from_numpy(quad.sub_q).cuda())
        box = torch.from_numpy(quad.box).cuda()
        return total.view(-1, 6) / (POROSITY * box[:, 3] * box[:, 4] * box[:, 5])[:, None], torch.from_numpy(quad.flags).cuda().long()
    vol = POROSITY * case["dx"] * case["dx"] * case["dz"]
    U = [torch.stack([g.qx[..., :-1], g.qx[..., 1:], g.qy[:, :-1], g.qy[:, 1:], g.qz[:-1], g.qz[1:]], dim=-1).view(-1, 6) for g in descs]
    return torch.cat(U) * (case["direction"] / vol), torch.cat([g.flags.reshape(-1) for g in descs]).long()


def exact(case, seed):
    """The floating outputs of `run` for the same inputs, in plain 64-bit torch arithmetic."""
    descs, quad, _, p = _inputs(case, seed)
    U, flags = _tables(case, descs, quad)
    n, ncell = case["n"], U.shape[0] // case["fields"]
    dims = torch.tensor([case["nx"], case["ny"], case["nz"]], device="cuda")
    stride = torch.tensor([1, case["nx"], case["nx"] * case["ny"]], device="cuda")
    size = torch.tensor([case["dx"], case["dx"], case["dz"]], dtype=torch.float64, device="cuda")
    end = torch.tensor(ENDS, dtype=torch.float64, device="cuda")
    t_max = case["t_max"] if case["t_max"] > 0 else HUGE_T
    stop_at_sink = case["kind"] != "transient"
    if quad is not None:
        off, nbs = (torch.from_numpy(a).cuda().long() for a in (quad.sub_off, quad.sub_nb))
        lo, hi = torch.from_numpy(quad.sub_lo).cuda(), torch.from_numpy(quad.sub_hi).cuda()
        box = torch.from_numpy(quad.box).cuda()

    def position(c, x):
        if quad is not None:
            return box[c, :3] + x * box[c, 3:]
        ijk = torch.stack([c % dims[0], (c // dims[0]) % dims[1], c // stride[2]], dim=1)
        return (ijk + x) * size

    x, t, c = torch.stack([p.xi, p.eta, p.zeta], dim=1), p.t.clone(), p.cell.long()
    if case["kind"] == "groups":
        offs, which = (torch.from_numpy(a).cuda() for a in _groups(case))
        g = which.long().repeat_interleave(offs[1:] - offs[:-1])
    elif case["kind"] == "transient":
        g = torch.searchsorted(end, t, right=True).clamp(max=len(ENDS) - 1)
    else:
        g = torch.zeros_like(c)
    snaps = case["snaps"]
    if snaps:
        times = torch.from_numpy(_snap_times(case)).cuda()
        rows = torch.full((n, snaps, 3), math.nan, dtype=torch.float64, device="cuda")
        ks = torch.searchsorted(times, t)
    zero = torch.zeros(n, dtype=torch.long, device="cuda")
    records = []
    ids = torch.arange(n, device="cuda")
    if stop_at_sink:
        ids = ids[(flags[g * ncell + c] & 2) == 0]
    while len(ids):
        xa, ta, ca, ga = x[ids], t[ids], c[ids], g[ids]
        u = U[ga * ncell + ca]
        u1, u2 = u[:, 0::2], u[:, 1::2]
        dts, A, up, e = _exit_times(u1, u2, xa)
        axis = torch.where(dts[:, 1] < dts[:, 0], 1, 0)
        dt = torch.minimum(dts[:, 0], dts[:, 1])
        axis = torch.where(dts[:, 2] < dt, 2, axis)
        dt = torch.minimum(dt, dts[:, 2])
        lim = torch.full_like(ta, t_max)
        if case["kind"] == "transient":
            lim = torch.minimum(lim, end[ga])
        stuck = torch.isinf(dt)
        at = (ta + dt > lim) | stuck
        tau = torch.where(at, lim - ta, dt)
        tau = torch.where(torch.isinf(tau), torch.zeros_like(tau), tau)
        if snaps:
            upto = torch.where(at, torch.searchsorted(times, lim, right=True), torch.searchsorted(times, ta + dt))
            cnt = (upto - ks[ids]).clamp(min=0)
            if int(cnt.sum()):
                rep = torch.repeat_interleave(torch.arange(len(ids), device="cuda"), cnt)
                which = ks[ids][rep] + torch.arange(len(rep), device="cuda") - (torch.cumsum(cnt, 0) - cnt)[rep]
                ds = torch.where(torch.isinf(lim[rep]) & stuck[rep], torch.zeros_like(lim[rep]), times[which] - ta[rep])[:, None]
                xs = (xa[rep] + (up[rep] * ds) * _psi(A[rep] * ds)).clamp(0.0, 1.0)
                rows[ids[rep], which] = position(ca[rep], xs)
                ks[ids] += cnt
        moved = (xa + (up * tau[:, None]) * _psi(A * tau[:, None])).clamp(0.0, 1.0)
        pick = torch.arange(3, device="cuda")[None] == axis[:, None]
        xn = torch.where(pick & ~at[:, None], e, moved)
        tn = torch.where(at, torch.where(torch.isinf(lim), ta, lim), ta + dt)
        t[ids] = tn
        x[ids] = xn
        if case["pathlines"]:
            records.append((ids[~at], tn[~at], position(ca, xn)[~at]))
        # at a limit: the next time step's field, or the end of the particle
        more = torch.zeros_like(at)
        if case["kind"] == "transient":
            more = at & (ga + 1 < len(ENDS)) & (lim < t_max)
            g[ids] = torch.where(more, ga + 1, ga)
        high = (e * pick).sum(1) > 0
        if quad is None:
            ijk = torch.stack([ca % dims[0], (ca // dims[0]) % dims[1], ca // stride[2]], dim=1)
            to = (ijk * pick).sum(1) + torch.where(high, 1, -1)
            inside = (to >= 0) & (to < dims[axis])
            cn = torch.where(inside, ca + torch.where(high, stride[axis], -stride[axis]), ca)
            enter = torch.where(pick, 1.0 - e, xn)
        else:
            f = 2 * axis + high.long()
            q0, q1 = off[6 * ca + f], off[6 * ca + f + 1]
            tangent = xn.gather(1, torch.stack([torch.where(axis == 0, 1, 0), torch.where(axis == 2, 1, 2)], dim=1))
            hit = q1 - 1
            for b in range(int((q1 - q0).max()) - 2, -1, -1):
                q = q0 + b
                ok = q < q1 - 1
                q = torch.where(ok, q, q1 - 1)
                hit = torch.where(ok & (lo[q] <= tangent).all(1) & (tangent <= hi[q]).all(1), q, hit)
            nb = torch.where(q1 > q0, nbs[hit], -1)
            inside = nb >= 0
            cn = torch.where(inside, nb, ca)
            same = (box[cn, :3] == box[ca, :3]) & (box[cn, 3:] == box[ca, 3:])
            mapped = ((box[ca, :3] + xn * box[ca, 3:] - box[cn, :3]) / box[cn, 3:]).clamp(0.0, 1.0)
            enter = torch.where(pick, 1.0 - e, torch.where(same, xn, mapped))
        go = ~at & inside
        c[ids] = torch.where(go, cn, ca)
        x[ids] = torch.where(go[:, None], enter, xn)
        live = go | more
        if stop_at_sink:
            live &= (flags[g[ids] * ncell + c[ids]] & 2) == 0
        if quad is not None:   # handed round a corner without moving: stopped
            zero[ids] = torch.where(go & (dt == 0), zero[ids] + 1, 0)
            live &= zero[ids] < 16
        ids = ids[live]
    final = dict(xi=x[:, 0], eta=x[:, 1], zeta=x[:, 2], t=t, xyz=position(c, x))
    if snaps:
        final["snap_xyz"] = rows
    if case["pathlines"]:
        ids, ts, xyz = (torch.cat(a) for a in zip(*records))
        o = torch.sort(ids, stable=True).indices
        m = min(len(o), _capacity(case))
        final.update(record_t=torch.zeros(_capacity(case), dtype=torch.float64, device="cuda"),
                     record_xyz=torch.zeros(_capacity(case), 3, dtype=torch.float64, device="cuda"))
        final["record_t"][:m] = ts[o][:m]
        final["record_xyz"][:m] = xyz[o][:m]
    if case["entry"] == "noalloc":
        order = ["counts"]
    elif case["pathlines"]:
        order = ["crossings", "dropped", "offsets", "record_t", "record_xyz", "record_cell", "record_face"]
    else:
        order = ["crossings"] + ([] if case["entry"] == "realisation" else ["tracked"])
    order += ["xi", "eta", "zeta", "t", "cell", "status", "ncross", "path_hash", "xyz"] + (["snap_xyz"] if snaps else [])
    return {k: final.get(k) for k in order}
