"""Sizes at which a call changes its route: results on both sides are those of the oracle."""
import numpy as np
import pytest

from workloads import configs as C

from . import test_gpu_pathline as L
from .gpu_util import compare, require_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pt():
    return require_gpu()


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
def test_staged_records_begin_above_a_wave_per_simd(pt, precision):
    """Up to 256 particles per compute unit the record pass writes each record where it belongs, one
    particle more and it stages them in LDS: the same records either way, and the oracle's (FP64)."""
    g = L.CASES["lognormal_wells"]()
    n = 256 * torch.cuda.get_device_properties(0).multi_processor_count
    p = C.release(np.random.Generator(np.random.PCG64(31)), n + 1, g.nx, g.ny, g.nz)
    kw = dict(schedule=1, sort=1, precision=precision)
    out, staged = L.gpu_pathlines(pt, [g], p, **kw)
    few, direct = L.gpu_pathlines(pt, [g], p.subset(np.arange(n)), **kw)
    m = int(direct["offsets"][-1])
    assert np.array_equal(staged["offsets"][:n + 1], direct["offsets"])
    for k in ("cell", "face", "t", "xyz"):
        assert np.array_equal(staged[k][:m], direct[k]), k
    assert out["summary"]["path_dropped"] == few["summary"]["path_dropped"] == 0
    if precision == 0:
        q = p.subset(np.arange(n - 700, n + 1))
        r, offs, flat = L.oracle_paths(g, q)
        first = int(staged["offsets"][n - 700])
        L.compare_paths(dict(offsets=staged["offsets"][n - 700:] - first, **{k: staged[k][first:] for k in ("cell", "face", "t", "xyz")}),
                        offs, flat, "staged")
        compare(out, r, idx=np.arange(n - 700, n + 1), label="staged", spacing=L.SP)


def test_grid_memory_is_reused(pt):
    """Grids loaded and released in turn take memory that earlier grids of other shapes held; every one
    gives the oracle's results, whether it was loaded from host or device arrays."""
    from oracle import oracle as O
    shapes = [(24, 17, 5), (24, 17, 5), (20, 19, 5), (9, 7, 3), (24, 17, 5), (31, 23, 6), (9, 7, 3)]
    for q, (nx, ny, nz) in enumerate(shapes):
        g = C.random_grid(nx, ny, nz, 1.5, 3.0, 500 + q, recharge=1e-3, porosity_field=bool(q % 2))
        p = C.release(np.random.Generator(np.random.PCG64(70 + q)), 777, nx, ny, nz)
        r = O.track(g, p)
        dev = type(g)(**{**vars(g), **{k: torch.from_numpy(np.ascontiguousarray(getattr(g, k))).cuda()
                                       for k in ("qx", "qy", "qz", "flags", "porosity") if getattr(g, k) is not None}})
        for kind in (g, dev):
            for layout in (1, 2):
                h = pt.pt_load_grid(kind)
                dp = pt.DeviceParticles.from_numpy(p, "cuda")
                xyz = torch.empty((p.n, 3), dtype=torch.float64, device="cuda")
                s = pt.track([h], dp, layout=layout, out_xyz=xyz)
                h.release()
                compare(dict(dp.to_numpy(), out_xyz=xyz.cpu().numpy(), summary=s), r, label="grid %d layout %d" % (q, layout),
                        spacing=(10.0, 10.0, 2.0))
