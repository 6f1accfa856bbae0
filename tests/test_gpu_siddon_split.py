"""Siddon back projection with four groups of threads that share the views: fewer views than groups, views that do not divide, rows closer
than a voxel and further apart, ragged tiles and chunks, against the oracle; an item's bits in any batch and on every call."""
import pytest

from synthetic import config, perturbed_poses, reduced, uniform_sinogram
from synthetic.configs import CONE, CONE_CURVED, PARALLEL
from tests.test_gpu_parity import TOL, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    return torch


def scan(geometry, pixel, nviews):
    par = geometry == PARALLEL
    return reduced(config(3), 8, nviews=nviews).replace(geom=geometry, nx=37, ny=34, nz=41, voxel_xy=1.0, voxel_z=1.0, nrows=int(75 / pixel) + 3,
                                                        ncols=int(95 / pixel), pixel_u=pixel, pixel_v=pixel, sod=0.0 if par else 150.0,
                                                        sdd=0.0 if par else 225.0, shift_u=0.3, shift_v=0.17, start_deg=3.0)


def check(torch_mod, oracle_mod, cfg):
    from paper_2307_05801_amd import Geometry
    geo = Geometry(cfg, model="siddon")
    print(f"[gpu] {cfg.geom} {cfg.nviews}: {geo.describe()}", flush=True)
    assert "+split" in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 9, batch=3)
    yt = torch_mod.from_numpy(y).cuda()
    out = geo.backproject(yt)
    for b in range(3):
        assert rel_l2(out[b].cpu().numpy(), oracle_mod.siddon.backproject(cfg, y[b])) <= TOL       # the parity tests' tolerance
        assert torch_mod.equal(out[b], geo.backproject(yt[b].contiguous()))
    assert torch_mod.equal(out, geo.backproject(yt))
    geo.close()


@pytest.mark.parametrize("geometry", [PARALLEL, CONE, CONE_CURVED])
@pytest.mark.parametrize("shape,pixel", [(0, 2.0), (1, 2.0), (1, 1.1)])
@pytest.mark.parametrize("nviews", [1, 3, 4, 10])
def test_views_shared_between_groups(torch_mod, oracle_mod, monkeypatch, geometry, shape, pixel, nviews):
    monkeypatch.setenv("LEAP_DEBUG", f"bp_split={shape}")
    check(torch_mod, oracle_mod, scan(geometry, pixel / 1.5 if geometry == PARALLEL else pixel, nviews))


@pytest.mark.parametrize("pixel", [1.3, 2.0])
def test_upright_modules(torch_mod, oracle_mod, pixel):
    check(torch_mod, oracle_mod, perturbed_poses(scan(CONE, pixel, 7), 3, shift_mm=2.0, upright=True))


@pytest.mark.parametrize("shape,pixel", [(0, 2.2), (1, 1.5)])
@pytest.mark.parametrize("nviews", [1, 2, 3, 9])
def test_tilted_modules(torch_mod, oracle_mod, monkeypatch, shape, pixel, nviews):
    monkeypatch.setenv("LEAP_DEBUG", f"bp_split={shape}")
    cfg = scan(CONE, pixel, nviews).replace(sod=180.0, sdd=270.0)
    check(torch_mod, oracle_mod, perturbed_poses(cfg, 3, shift_mm=2.0, tilt_rad=0.05))


@pytest.mark.parametrize("kind", ["parallel", "cone", "upright", "tilted"])
def test_batches_of_every_size(torch_mod, oracle_mod, kind):
    """A batch that fills the chip takes another kernel than one volume: the same sums in another order, to the last bits."""
    from paper_2307_05801_amd import Geometry
    cfg = scan(PARALLEL if kind == "parallel" else CONE, 1.5 if kind == "parallel" else 2.2, 8).replace(nx=80, ny=77, nz=64, nrows=60, ncols=100)
    if kind != "parallel":
        cfg = cfg.replace(sod=400.0, sdd=600.0)
    if kind in ("upright", "tilted"):
        cfg = perturbed_poses(cfg, 3, shift_mm=2.0, upright=kind == "upright", **({} if kind == "upright" else {"tilt_rad": 0.05}))
    geo = Geometry(cfg, model="siddon")
    print(f"[gpu] {kind}: {geo.describe()}", flush=True)
    assert "+split" in geo.describe(), geo.describe()
    y = torch_mod.from_numpy(uniform_sinogram(cfg, 9, batch=17)).cuda()
    alone = torch_mod.stack([geo.backproject(y[b].contiguous()) for b in range(17)])
    assert rel_l2(alone[16].cpu().numpy(), oracle_mod.siddon.backproject(cfg, y[16].cpu().numpy())) <= TOL
    for batch in (1, 2, 8, 17):
        out = geo.backproject(y[:batch].contiguous())
        assert torch_mod.equal(out, geo.backproject(y[:batch].contiguous())), batch
        for b in range(batch):                              # sums of eight views' shares in two orders: 8 * 2^-24 at most
            assert float((out[b] - alone[b]).norm()) <= 5e-7 * float(alone[b].norm()), (batch, b)
    geo.close()
