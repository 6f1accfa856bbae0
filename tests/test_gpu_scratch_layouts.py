"""One handle, batches of different sizes: the scratch copy is laid out differently for each, and a call must not read what an
earlier one left between its columns."""
import pytest

from synthetic import CTConfig, perturbed_poses
from synthetic.configs import CONE, PARALLEL

pytestmark = pytest.mark.gpu


def scan(name, geom=CONE, nrows=40):
    par = dict(sod=0.0, sdd=0.0) if geom == PARALLEL else dict(sod=150.0, sdd=225.0)
    return CTConfig(name, geom, nviews=7, arc_deg=360.0, nrows=nrows, ncols=96, pixel_v=1.5, pixel_u=1.6, nx=50, ny=70, nz=20, voxel_xy=1.0,
                    voxel_z=1.0, start_deg=3.0, **par)


SCANS = [(scan("cone_one_row_per_lane"), "siddon"), (scan("parallel_one_row_per_lane", PARALLEL), "siddon"),
         (scan("pairs", nrows=90), "siddon"), (perturbed_poses(scan("upright"), 5, shift_mm=4.0, upright=True), "siddon"),
         (perturbed_poses(scan("tilted"), 5, shift_mm=4.0, tilt_rad=0.1), "siddon"), (scan("footprint"), "sf"),
         (scan("footprint_rows", PARALLEL), "sf")]


@pytest.mark.parametrize("cfg,model", SCANS, ids=lambda v: getattr(v, "name", v))
def test_layouts_of_other_batches_leave_nothing_behind(cfg, model):
    import torch
    from paper_2307_05801_amd import Geometry
    used = Geometry(cfg, model=model)
    print(f"[gpu] {cfg.name}: {used.describe()}", flush=True)
    assert "A=columns" in used.describe(), used.describe()
    for batch in (1, 16, 5, 16, 1, 2):
        x = 1.0 + torch.rand((batch,) + used.vol_shape, device="cuda")
        fresh = Geometry(cfg, model=model)
        assert torch.equal(used.project(x), fresh.project(x)), batch
        fresh.close()
    used.close()
