"""Footprints on tilted modules through the tiled kernels (md_footprint_tiled.h) against the oracle: edges of the voxel tiles
(16 x 16 of 8, 2 or 1) and of the detector tiles (16 x 64), footprints wider and taller than the three columns and rows of the common
case, modules turned by a quarter, and values a weight of zero must not spread."""
import numpy as np
import pytest

from synthetic import CTConfig, perturbed_poses, uniform_sinogram, uniform_volume
from synthetic.configs import CONE, modular_from

pytestmark = pytest.mark.gpu

TOL = 6e-8          # sums in double precision, every output rounded to float32 once: at most 2^-24 of it


def scan(nx, ny, nz, nrows, ncols, nviews=5, pixel_u=1.5, pixel_v=1.5, voxel_z=1.0, tilt=0.1, seed=3, **kw):
    base = CTConfig(f"tilted_{nx}x{ny}x{nz}_{nrows}x{ncols}_{pixel_u}", CONE, nviews=nviews, arc_deg=360.0, nrows=nrows, ncols=ncols,
                    pixel_v=pixel_v, pixel_u=pixel_u, nx=nx, ny=ny, nz=nz, voxel_xy=1.0, voxel_z=voxel_z, sod=160.0, sdd=240.0, shift_u=0.4,
                    shift_v=-0.3, center_x=1.0, center_y=-2.0, center_z=0.5, start_deg=3.0).replace(**kw)
    return perturbed_poses(base, seed, shift_mm=4.0, tilt_rad=tilt)


def rolled(angle):
    """Modules turned about their normals; by a quarter, a voxel's in-plane corners fall on one column and it has no footprint."""
    base = modular_from(scan(20, 24, 30, 50, 40).replace(geom=CONE, poses=None))
    co, si = (0.0, 1.0) if angle == "quarter" else (np.cos(angle), np.sin(angle))
    poses = tuple(p[:6] + tuple(co * u + si * v for u, v in zip(p[6:9], p[9:12])) + tuple(co * v - si * u for u, v in zip(p[6:9], p[9:12]))
                  for p in base.poses)
    return base.replace(name=f"rolled_{angle}", poses=poses)


SCANS = [scan(1, 1, 1, 3, 2), scan(16, 16, 8, 64, 16), scan(17, 15, 9, 65, 17), scan(33, 40, 23, 40, 63, tilt=0.5),
         scan(24, 24, 60, 130, 70, pixel_v=0.9), scan(9, 8, 12, 90, 60, pixel_u=0.42, pixel_v=0.45), scan(30, 30, 10, 20, 24, pixel_u=4.0, pixel_v=3.5),
         scan(18, 20, 11, 60, 50, voxel_z=2.3, pixel_v=1.1), scan(80, 79, 105, 60, 50), scan(47, 48, 81, 40, 40), scan(47, 48, 79, 40, 40), rolled(1.2), rolled(2.9), rolled("quarter")]


@pytest.mark.parametrize("cfg", SCANS, ids=lambda c: c.name)
def test_tiled_kernels_match_oracle(oracle_mod, cfg):
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(cfg)
    print(f"[gpu] {cfg.name}: {geo.describe()}", flush=True)
    assert "A=general(tiles)" in geo.describe() and "AT=general(tiled)" in geo.describe(), geo.describe()
    x, y = uniform_volume(cfg, 3, batch=2), uniform_sinogram(cfg, 4, batch=2)
    xt, yt = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    ax, aty = geo.project(xt), geo.backproject(yt)
    for _ in range(3):
        assert torch.equal(geo.project(xt), ax) and torch.equal(geo.backproject(yt), aty)
    for got, want in ((ax[1].cpu().numpy(), oracle_mod.project(cfg, x[1])), (aty[1].cpu().numpy(), oracle_mod.backproject(cfg, y[1]))):
        # (+ what knots rounded in double leave of a footprint without width: 1e-15 pixels a weight, a few thousand weights)
        assert np.linalg.norm(got - want) <= TOL * np.linalg.norm(want) + 1e-12
        assert np.abs(got - want).max() <= 2e-7 * np.abs(want).max() + 1e-12
    geo.close()


# back projections of few views or many tiles: eight, four and two voxels per thread, four groups of four and of two
SHAPES = [scan(130, 140, 90, 40, 60, nviews=2), scan(80, 79, 105, 60, 50, nviews=2), scan(51, 60, 81, 80, 50, nviews=9), scan(40, 41, 101, 60, 40, nviews=3),
          scan(48, 47, 51, 60, 50, nviews=17)]


@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: c.name)
def test_every_shape_of_the_back_projection_matches_oracle(oracle_mod, cfg):
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(cfg)
    print(f"[gpu] {cfg.name}: {geo.describe()}", flush=True)
    assert "AT=general(tiled)" in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 4)[0]
    yt = torch.from_numpy(y).cuda()
    got = geo.backproject(yt)
    assert torch.equal(geo.backproject(yt), got)
    got, want = got.cpu().numpy(), oracle_mod.backproject(cfg, y)
    assert np.linalg.norm(got - want) <= TOL * np.linalg.norm(want) + 1e-12
    assert np.abs(got - want).max() <= 2e-7 * np.abs(want).max() + 1e-12
    geo.close()


def test_a_weight_of_zero_spreads_nothing():
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(SCANS[3])
    x, y = torch.rand(geo.vol_shape, device="cuda"), torch.rand(geo.sino_shape, device="cuda")
    ax, aty = geo.project(x), geo.backproject(y)
    w, r = torch.zeros_like(x), torch.zeros_like(y)
    w[12, 20, 17], r[2, 21, 30] = 1.0, 1.0
    hit_rays, hit_voxels = geo.project(w) > 0, geo.backproject(r) > 0
    x[12, 20, 17], y[2, 21, 30] = float("inf"), float("nan")
    axb, atyb = geo.project(x), geo.backproject(y)
    assert torch.equal(~axb.isfinite(), hit_rays) and torch.allclose(axb[~hit_rays], ax[~hit_rays], rtol=1e-6)
    assert torch.equal(atyb.isnan(), hit_voxels) and torch.allclose(atyb[~hit_voxels], aty[~hit_voxels], rtol=1e-6)
    geo.close()


# 1, 2 and 4 voxels per thread with the views shared by four groups of threads; 1, 4 and 8 with none; four waves per detector tile (780 tiles)
SHAPES = [scan(20, 24, 10, 30, 40, nviews=9), scan(47, 48, 38, 50, 70, nviews=10), scan(64, 62, 51, 60, 70, nviews=7), scan(20, 24, 10, 31, 40, nviews=1),
          scan(96, 90, 76, 64, 100, nviews=2), scan(128, 126, 102, 70, 120, nviews=2), scan(20, 24, 10, 60, 200, nviews=60)]


@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: f"{c.name}_{c.nviews}")
def test_views_and_layers_shared(oracle_mod, cfg):
    test_tiled_kernels_match_oracle(oracle_mod, cfg)
