"""Footprint back projection with two volumes per workgroup: a volume and its mirror image about the source plane, two items of a batch.

Odd and even layers and rows (the middle layer is its own mirror image), ragged tiles and chunks, every window shape, parallel, flat
and cylindrical detectors, against the oracle; off-centre detectors and volumes, which are not mirrored; batches bit for bit."""
import pytest

from synthetic import config, reduced, uniform_sinogram
from synthetic.configs import CONE, CONE_CURVED, PARALLEL
from tests.test_gpu_parity import TOL, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    return torch


def scan(geometry, nz, nrows, pixel, nx=37, ny=34, **kw):
    par = geometry == PARALLEL
    return reduced(config(3), 8, nviews=10).replace(geom=geometry, nx=nx, ny=ny, nz=nz, voxel_xy=1.0, voxel_z=1.0, nrows=nrows,
                                                    ncols=61, pixel_u=pixel, pixel_v=pixel, sod=0.0 if par else 150.0, sdd=0.0 if par else 225.0,
                                                    shift_u=0.3, **kw)


SIZES = [(9, 16), (40, 50), (41, 50), (41, 51), (70, 73), (131, 128)]
# pixel (mm, at the detector) and window shape; the wide windows, for voxels of three columns and more, on diverging beams
CASES = [(g, nz, nrows, pixel, shape) for g in (PARALLEL, CONE, CONE_CURVED) for nz, nrows in SIZES for pixel, shape in ((2.4, 0), (1.8, 1), (2.4, 2))]
CASES += [(g, nz, nrows, 1.2, 3) for g in (CONE, CONE_CURVED) for nz, nrows in SIZES[:5]]


@pytest.mark.parametrize("geometry,nz,nrows,pixel,shape", CASES)
def test_mirror_image(torch_mod, oracle_mod, monkeypatch, geometry, nz, nrows, pixel, shape):
    from paper_2307_05801_amd import Geometry
    if geometry == PARALLEL:
        pixel /= 1.5
    monkeypatch.setenv("LEAP_DEBUG", f"bp_pair={shape},bp_split=-1")
    cfg = scan(geometry, nz, nrows, pixel)
    geo = Geometry(cfg)
    assert "+mirror" in geo.describe(), geo.describe()
    print(f"[gpu] {geometry} {nz} {nrows} {pixel}: {geo.describe()}", flush=True)
    y = uniform_sinogram(cfg, 7, batch=2)
    yt = torch_mod.from_numpy(y).cuda()
    out = geo.backproject(yt)
    for b in range(2):
        assert rel_l2(out[b].cpu().numpy(), oracle_mod.backproject(cfg, y[b])) <= TOL      # the parity tests' tolerance
        assert torch_mod.equal(out[b], geo.backproject(yt[b].contiguous()))
    geo.close()


@pytest.mark.parametrize("geometry", [CONE, CONE_CURVED])
@pytest.mark.parametrize("off", [dict(shift_v=0.25), dict(center_z=1.5)])
def test_no_mirror_image_off_centre(torch_mod, oracle_mod, monkeypatch, geometry, off):
    """Two items per workgroup instead, the same bits as alone whatever the batch."""
    from paper_2307_05801_amd import Geometry
    cfg = scan(geometry, 40, 50, 1.4, nx=151, ny=149, **off).replace(sod=600.0, sdd=900.0, ncols=220, pixel_u=1.2)
    monkeypatch.setenv("LEAP_DEBUG", "bp_split=-1")
    geo = Geometry(cfg)
    assert "+pairs" in geo.describe(), geo.describe()
    print(f"[gpu] {off}: {geo.describe()}", flush=True)
    assert "+mirror" not in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 8, batch=9)
    yt = torch_mod.from_numpy(y).cuda()
    out = geo.backproject(yt)                 # eight in twos, one by itself
    for b in (0, 8):
        assert rel_l2(out[b].cpu().numpy(), oracle_mod.backproject(cfg, y[b])) <= TOL
    for batch in (1, 2, 8):
        got = geo.backproject(yt[:batch].contiguous())
        assert torch_mod.equal(out[:batch], got), batch
    geo.close()


def test_a_sample_that_is_not_finite_stays_in_its_half(torch_mod):
    """A voxel and its mirror image share weights, not samples."""
    from paper_2307_05801_amd import Geometry
    cfg = scan(CONE, 256, 280, 2.0, nx=150, ny=150).replace(sod=500.0, sdd=750.0)
    geo = Geometry(cfg)
    assert "+mirror" in geo.describe(), geo.describe()
    y = torch_mod.rand(cfg.sino_shape, device="cuda")
    ref = geo.backproject(y)
    y[3, 200, 30] = float("inf")
    out = geo.backproject(y)
    assert torch_mod.equal(out[:128], ref[:128])
    assert bool((~out[128:].isfinite()).any())
    geo.close()


@pytest.mark.parametrize("geometry", [PARALLEL, CONE, CONE_CURVED])
@pytest.mark.parametrize("shape,pixel", [(0, 2.4), (1, 1.8), (2, 1.8), (2, 1.2)])
@pytest.mark.parametrize("nviews", [1, 3, 4, 10])
@pytest.mark.parametrize("shift_v", [0.0, 0.25])
def test_views_shared_between_groups(torch_mod, oracle_mod, monkeypatch, geometry, shape, pixel, nviews, shift_v):
    """Fewer views than groups, views that do not divide; the mirror image and two items; an item's bits in any batch."""
    from paper_2307_05801_amd import Geometry
    if geometry == PARALLEL:
        pixel /= 1.5
    monkeypatch.setenv("LEAP_DEBUG", f"bp_split={shape}")
    cfg = scan(geometry, 41, 51, pixel).replace(nviews=nviews, shift_v=shift_v)
    geo = Geometry(cfg)
    print(f"[gpu] {geometry} {nviews}: {geo.describe()}", flush=True)
    assert "+split" in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 9, batch=3)
    yt = torch_mod.from_numpy(y).cuda()
    out = geo.backproject(yt)
    for b in range(3):
        assert rel_l2(out[b].cpu().numpy(), oracle_mod.backproject(cfg, y[b])) <= TOL
        assert torch_mod.equal(out[b], geo.backproject(yt[b].contiguous()))
    assert torch_mod.equal(out, geo.backproject(yt))
    geo.close()


def test_views_shared_on_upright_modules(torch_mod, oracle_mod):
    from paper_2307_05801_amd import Geometry
    from synthetic import perturbed_poses
    cfg = perturbed_poses(scan(CONE, 33, 40, 2.0), 3, shift_mm=2.0, upright=True)
    geo = Geometry(cfg)
    assert "+split" in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 4, batch=2)
    yt = torch_mod.from_numpy(y).cuda()
    out = geo.backproject(yt)
    for b in range(2):
        assert rel_l2(out[b].cpu().numpy(), oracle_mod.backproject(cfg, y[b])) <= TOL
        assert torch_mod.equal(out[b], geo.backproject(yt[b].contiguous()))
    geo.close()


@pytest.mark.parametrize("geometry", [PARALLEL, CONE, CONE_CURVED])
@pytest.mark.parametrize("shift_v", [0.0, 0.25])
def test_batches_of_every_size(torch_mod, oracle_mod, geometry, shift_v):
    """A batch that fills the chip takes another kernel than one volume: the same sums in another order, to the last bits."""
    from paper_2307_05801_amd import Geometry
    cfg = scan(geometry, 64, 70, 2.0 / 1.5 if geometry == PARALLEL else 2.0, nx=96, ny=93).replace(nviews=8, ncols=130, shift_v=shift_v)
    if geometry != PARALLEL:
        cfg = cfg.replace(sod=400.0, sdd=600.0)
    geo = Geometry(cfg)
    print(f"[gpu] {geometry} {shift_v}: {geo.describe()}", flush=True)
    assert "+split" in geo.describe(), geo.describe()
    y = torch_mod.from_numpy(uniform_sinogram(cfg, 9, batch=17)).cuda()
    alone = torch_mod.stack([geo.backproject(y[b].contiguous()) for b in range(17)])
    assert rel_l2(alone[16].cpu().numpy(), oracle_mod.backproject(cfg, y[16].cpu().numpy())) <= TOL
    for batch in (1, 2, 3, 8, 15, 17):                      # (the seventeenth item is a launch of its own)
        out = geo.backproject(y[:batch].contiguous())
        assert torch_mod.equal(out, geo.backproject(y[:batch].contiguous())), batch
        for b in range(batch):                              # sums of eight views' shares in two orders: 8 * 2^-24 at most
            assert float((out[b] - alone[b]).norm()) <= 5e-7 * float(alone[b].norm()), (batch, b)
    geo.close()


# pair shape, the one-volume shape of the same height, pixel (voxels at the axis)
@pytest.mark.parametrize("pair,single,pixel", [(0, 1, 2.4), (1, 2, 1.9), (2, 3, 2.4), (3, 4, 1.3)])
@pytest.mark.parametrize("geometry", [PARALLEL, CONE, CONE_CURVED])
@pytest.mark.parametrize("voxel_z", [0.7, 1.0, 1.35])
def test_two_items_of_every_shape(torch_mod, oracle_mod, monkeypatch, geometry, pair, single, pixel, voxel_z):
    """Off centre, voxels of up to one row and of up to two: two items per workgroup give the bits of one per workgroup, and the same on
    every call (256 threads stage a window of 51 columns with one to spare)."""
    from paper_2307_05801_amd import Geometry
    cfg = scan(geometry, 41, 51, pixel / 1.5 if geometry == PARALLEL else pixel, shift_v=0.25).replace(voxel_z=voxel_z)
    monkeypatch.setenv("LEAP_DEBUG", f"bp_pair={pair},bp_shape={single}")
    geo = Geometry(cfg)
    print(f"[gpu] {geometry} {pair} {voxel_z}: {geo.describe()}", flush=True)
    if geometry == PARALLEL and pair == 3:
        assert "tiled(" in geo.describe(), geo.describe()          # (three columns and more: diverging beams)
    else:
        assert "+pairs" in geo.describe() and "+split" not in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 8, batch=5)
    yt = torch_mod.from_numpy(y).cuda()
    out = geo.backproject(yt)
    for b in (0, 3):
        assert rel_l2(out[b].cpu().numpy(), oracle_mod.backproject(cfg, y[b])) <= TOL
    for b in range(5):
        assert torch_mod.equal(out[b], geo.backproject(yt[b].contiguous())), b
    for _ in range(6):
        assert torch_mod.equal(out, geo.backproject(yt))
    geo.close()
