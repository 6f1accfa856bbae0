"""Forward projection, footprint model: the row-height classes and two volumes per wave.

Rows of every class (up to half a voxel, a voxel, a voxel and a half, two, three) and scans whose rows change class from voxel
column to voxel column, against the oracle; batches of two, three and five items, bit for bit what each item gives alone."""
import pytest

from synthetic import config, reduced, uniform_volume
from tests.test_gpu_parity import TOL, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    return torch


def scan(pixel_v, nrows, nz, **kw):
    """32 x 30 x nz voxels of 1 mm at magnifications 1.27 to 1.79; pixel_v / 1.5: voxels per row at the axis."""
    return reduced(config(3), 8, nviews=9).replace(nx=32, ny=30, nz=nz, voxel_xy=1.0, voxel_z=1.0, nrows=nrows, ncols=45, pixel_u=1.5, pixel_v=pixel_v,
                                                   sod=100.0, sdd=150.0, shift_v=0.2, shift_u=-0.3, **kw)


@pytest.mark.parametrize("pixel_v,nrows", [(0.6, 97), (0.75, 64), (1.2, 65), (1.5, 40), (1.8, 33), (2.25, 36), (2.6, 32), (3.0, 33), (3.55, 32)])
@pytest.mark.parametrize("cw", ["cw=2", "cw=4"])
def test_rows_of_every_height(torch_mod, oracle_mod, monkeypatch, pixel_v, nrows, cw):
    from paper_2307_05801_amd import Geometry
    monkeypatch.setenv("LEAP_DEBUG", cw + ",pairs=1")        # two volumes per wave however few the waves, where there is a kernel for two
    cfg = scan(pixel_v, nrows, 40)
    geo = Geometry(cfg)
    print(f"[gpu] pixel_v={pixel_v}: {geo.describe()}", flush=True)
    assert "A=columns" in geo.describe() and (pixel_v > 0.6 or "nkp=2" in geo.describe()), geo.describe()
    x = uniform_volume(cfg, 5, batch=5)
    xt = torch_mod.from_numpy(x).cuda()
    y = geo.project(xt)
    # float sums of products whose positions are double: the parity tests' tolerance
    assert rel_l2(y[0].cpu().numpy(), oracle_mod.project(cfg, x[0])) <= TOL
    assert rel_l2(y[3].cpu().numpy(), oracle_mod.project(cfg, x[3])) <= TOL
    for b in range(5):
        assert torch_mod.equal(y[b], geo.project(xt[b].contiguous())), b
    for batch in (2, 3):
        assert torch_mod.equal(y[:batch], geo.project(xt[:batch].contiguous())), batch
    geo.close()


@pytest.mark.parametrize("debug", ["pairs=1", "pairs=1,slab=8"])
@pytest.mark.parametrize("geometry", ["cone", "curved", "upright"])
@pytest.mark.parametrize("pixel_v,nrows", [(1.4, 97), (1.3, 200), (2.2, 300), (1.4, 500), (2.8, 97), (2.6, 140), (3.5, 97)])
def test_two_volumes_per_wave(torch_mod, oracle_mod, monkeypatch, geometry, pixel_v, nrows, debug):
    """One to four groups of rows (four of one volume, two at a time of two), the cylinder's and the upright modules' kernels,
    a volume that goes through in slabs and adds to what earlier slabs left: every item bit for bit what it gives alone."""
    from paper_2307_05801_amd import Geometry
    from synthetic import perturbed_poses
    from synthetic.configs import CONE_CURVED
    cfg = scan(pixel_v, nrows, 24).replace(nx=19, ny=22, nviews=5)
    cfg = cfg.replace(geom=CONE_CURVED) if geometry == "curved" else cfg
    cfg = perturbed_poses(cfg, 4, shift_mm=2.0, upright=True) if geometry == "upright" else cfg
    x = uniform_volume(cfg, 5, batch=5)
    xt = torch_mod.from_numpy(x).cuda()
    monkeypatch.setenv("LEAP_DEBUG", debug.replace("pairs=1", "pairs=0"))
    alone = Geometry(cfg)
    monkeypatch.setenv("LEAP_DEBUG", debug)
    geo = Geometry(cfg)
    print(f"[gpu] {geometry} {pixel_v} {nrows} {debug}: {geo.describe()}", flush=True)
    assert "A=columns" in geo.describe(), geo.describe()
    y = alone.project(xt)
    for b in (0, 4):
        assert rel_l2(y[b].cpu().numpy(), oracle_mod.project(cfg, x[b])) <= TOL
    for batch in (2, 3, 5):
        assert torch_mod.equal(y[:batch], geo.project(xt[:batch].contiguous())), batch
    geo.close()
    alone.close()
