"""Footprint back projection under the 42-column window, whose width does not divide the workgroup (four of 256 threads stage
nothing), against the oracle: flat, cylindrical and upright-modular detectors, two- and three-row footprints three and four columns
wide, ragged volumes, pixel heights that are no short binary fractions, batches; the same bits on every call."""
import numpy as np
import pytest

from synthetic import CTConfig, perturbed_poses, uniform_sinogram
from synthetic.configs import CONE, CONE_CURVED

pytestmark = pytest.mark.gpu

TOL = 2e-6           # float32 sums of a few hundred products of weights good to a few units of 2^-24


PIXEL_U = {"flat": {3: 1.37, 4: 1.23}, "curved": {3: 1.27, 4: 1.13}, "upright": {3: 1.57, 4: 1.37}}
PIXEL_V = {"flat": {2: 1.73, 3: 1.57}, "curved": {2: 1.73, 3: 1.57}, "upright": {2: 1.93, 3: 1.73}}


def scan(name, nc, nv, kind, nx=37, ny=50, nz=41, nviews=40):
    geom, pixel_u, pixel_v = CONE_CURVED if kind == "curved" else CONE, PIXEL_U[kind][nc], PIXEL_V[kind][nv]
    return CTConfig(name, geom, nviews=nviews, arc_deg=360.0, nrows=93, ncols=131, pixel_v=pixel_v, pixel_u=pixel_u, nx=nx, ny=ny, nz=nz,
                    voxel_xy=1.0, voxel_z=1.0, sod=160.0, sdd=214.0, shift_u=0.4, shift_v=-0.3, center_x=1.0, center_y=-2.0, center_z=0.5,
                    start_deg=3.0)


SCANS = [(f"{kind}_{nc}_{nv}", nc, nv, kind) for kind in ("flat", "curved", "upright") for nc in (3, 4) for nv in (2, 3)]


@pytest.mark.parametrize("name,nc,nv,kind", SCANS, ids=lambda v: v if isinstance(v, str) else "")
def test_wide_window_matches_oracle_and_repeats(oracle_mod, name, nc, nv, kind, monkeypatch):
    import torch
    from paper_2307_05801_amd import Geometry
    cfg = scan(name, nc, nv, kind)
    if kind == "upright":
        cfg = perturbed_poses(cfg, 4, shift_mm=3.0, upright=True)
    monkeypatch.setenv("LEAP_DEBUG", "bp_shape=6")
    geo = Geometry(cfg)
    print(f"[gpu] {cfg.name}: {geo.describe()}", flush=True)
    assert f"AT=tiled(nc={nc},nv={nv},zc=32,wide" in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 4, batch=3)
    yt = torch.from_numpy(y).cuda()
    out = geo.backproject(yt)
    for _ in range(8):
        assert torch.equal(geo.backproject(yt), out)
    got = out.cpu().numpy()
    for b in (0, 2):
        want = oracle_mod.backproject(cfg, y[b])
        assert np.linalg.norm(got[b] - want) <= TOL * np.linalg.norm(want)
        assert np.abs(got[b] - want).max() <= 2e-5 * np.abs(want).max()
    geo.close()
