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
    monkeypatch.setenv("LEAP_DEBUG", cw)
    cfg = scan(pixel_v, nrows, 40)
    geo = Geometry(cfg)
    print(f"[gpu] pixel_v={pixel_v}: {geo.describe()}", flush=True)
    assert "A=columns" in geo.describe(), geo.describe()
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

