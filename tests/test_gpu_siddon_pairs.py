"""Siddon forward projection, two adjacent rows per lane (sd_project_pairs), against the oracle: remainders of 128-row bands and
of four-column workgroups, rows closer than a voxel, further apart, and on either side of one voxel within a scan, level rays,
modules with their own source heights, volumes walked in narrow slabs."""
import numpy as np
import pytest

from synthetic import CTConfig, perturbed_poses, uniform_sinogram, uniform_volume
from synthetic.configs import CONE, CONE_CURVED, PARALLEL

pytestmark = pytest.mark.gpu

# float32 sums of a few hundred lengths; a length's share is a fraction of a voxel, exact to 2^-32, over the ray's rise
TOL = 2e-6


def scan(name, nrows, ncols, pixel_v, nx=61, ny=70, nz=57, geom=CONE, nviews=7, **kw):
    base = CTConfig(name, geom, nviews=nviews, arc_deg=360.0, nrows=nrows, ncols=ncols, pixel_v=pixel_v, pixel_u=1.4, nx=nx, ny=ny, nz=nz,
                    voxel_xy=1.0, voxel_z=1.0, sod=150.0, sdd=225.0, shift_u=0.27, shift_v=-0.31, center_x=1.0, center_y=-2.0, center_z=0.5,
                    start_deg=3.0)
    return base.replace(**kw)


SCANS = [scan("rows65", 65, 77, 1.5), scan("rows128", 128, 64, 0.7), scan("rows129", 129, 81, 0.9), scan("rows300", 300, 33, 0.35),
         scan("apart", 70, 90, 2.0), scan("either_side", 90, 60, 1.45), scan("one_column", 66, 1, 1.5),
         scan("level", 80, 95, 0.8, geom=PARALLEL, sod=0.0, sdd=0.0, pixel_u=1.0),
         scan("level_on_faces", 70, 95, 1.0, geom=PARALLEL, sod=0.0, sdd=0.0, pixel_u=1.0, shift_v=0.5, nz=56, center_z=0.0),
         scan("curved", 100, 80, 1.2, geom=CONE_CURVED), perturbed_poses(scan("upright", 96, 70, 1.6), 5, shift_mm=6.0, upright=True)]


@pytest.mark.parametrize("slab", ["", "slab=8"])
@pytest.mark.parametrize("cfg", SCANS, ids=lambda c: c.name)
def test_two_rows_per_lane_match_oracle(oracle_mod, cfg, slab, monkeypatch):
    import torch
    from paper_2307_05801_amd import Geometry
    oracle_mod.siddon.build()
    if slab:
        monkeypatch.setenv("LEAP_DEBUG", slab)
    geo = Geometry(cfg, model="siddon")
    print(f"[gpu] {cfg.name}: {geo.describe()}", flush=True)
    assert "A=columns(" in geo.describe() and "pairs" in geo.describe(), geo.describe()
    x = uniform_volume(cfg, 3, batch=2)
    got = geo.project(torch.from_numpy(x).cuda()).cpu().numpy()
    for b in range(2):
        want = oracle_mod.siddon.project(cfg, x[b])
        assert np.linalg.norm(got[b] - want) <= TOL * np.linalg.norm(want)
        assert np.abs(got[b] - want).max() <= 2e-5 * np.abs(want).max()
    geo.close()


# an odd detector over a volume of even height: the middle row runs along a z-face and belongs to the voxels above it
FACE = dict(nx=30, ny=28, nz=24, shift_v=0.0, center_z=0.0)
FLAT_BEAM = dict(FACE, geom=PARALLEL, sod=0.0, sdd=0.0)
FACES = [scan("parallel_on_face", 67, 60, 0.75, **FLAT_BEAM), scan("parallel_near_face", 67, 60, 0.7, **FLAT_BEAM),
         scan("parallel_below_face", 131, 60, 0.35, **FLAT_BEAM), scan("parallel_short", 45, 60, 0.9, **FLAT_BEAM),
         scan("parallel_on_face_apart", 69, 60, 1.25, **dict(FLAT_BEAM, nz=60)), scan("cone_on_face", 67, 60, 0.75, **FACE),
         scan("cone_near_face", 67, 60, 0.7, **FACE), scan("cone_below_face", 67, 60, 0.85, **FACE)]


@pytest.mark.parametrize("cfg", FACES, ids=lambda c: c.name)
def test_rows_on_a_face_match_oracle(oracle_mod, cfg):
    import torch
    from paper_2307_05801_amd import Geometry
    oracle_mod.siddon.build()
    geo = Geometry(cfg, model="siddon")
    print(f"[gpu] {cfg.name}: {geo.describe()}", flush=True)
    assert "A=columns" in geo.describe() and "AT=tiled" in geo.describe(), geo.describe()
    x, y = uniform_volume(cfg, 3, batch=2), uniform_sinogram(cfg, 4, batch=2)
    ax = geo.project(torch.from_numpy(x).cuda()).cpu().numpy()
    aty = geo.backproject(torch.from_numpy(y).cuda()).cpu().numpy()
    for got, want in ((ax[1], oracle_mod.siddon.project(cfg, x[1])), (aty[1], oracle_mod.siddon.backproject(cfg, y[1]))):
        assert np.linalg.norm(got - want) <= TOL * np.linalg.norm(want)
        assert np.abs(got - want).max() <= 2e-5 * np.abs(want).max()
    geo.close()


def test_voxels_a_level_ray_does_not_meet_add_nothing(oracle_mod):
    """Layers of 1e8 beside layers of about 1: rows that run in the latter see nothing of the former."""
    import torch
    from paper_2307_05801_amd import Geometry
    oracle_mod.siddon.build()
    cfg = scan("contrast", 80, 60, 1.0, nx=30, ny=28, nz=60, geom=PARALLEL, sod=0.0, sdd=0.0, shift_v=0.0, center_z=0.0)
    x = 1.0 + uniform_volume(cfg, 3)
    x[:, ::2] = 1e8
    geo = Geometry(cfg, model="siddon")
    assert "pairs" in geo.describe(), geo.describe()
    got = geo.project(torch.from_numpy(x).cuda()).cpu().numpy()[0]
    want = oracle_mod.siddon.project(cfg, x[0])
    light = want.max(axis=(0, 2)) < 1e4
    assert light.sum() >= 40
    assert np.abs(got - want)[:, light].max() <= 2e-5 * want[:, light].max()
    geo.close()
