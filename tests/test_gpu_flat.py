"""Flat scans (one detector row, one voxel layer): the kernels of sf_flat.h against the oracle, at the edges of their tiles
(8 x 8 voxels, 64 columns), of their splits over waves and of their groups of items."""
import numpy as np
import pytest

from synthetic import CTConfig, uniform_sinogram, uniform_volume
from synthetic.configs import FAN, PARALLEL

pytestmark = pytest.mark.gpu

# float32 sums of up to 3 * 200 products whose weights carry a few units of 2^-24 each: sqrt(600) * 2^-25 + 4 * 2^-24 = 1e-6
TOL = 2e-6


def scan(geom, nx, ny, ncols, nviews, pixel_u=1.3, **kw):
    fan = dict(sod=400.0, sdd=700.0) if geom == FAN else {}
    return CTConfig(f"flat_{geom}_{nx}x{ny}_{ncols}_{nviews}", geom, nviews=nviews, arc_deg=360.0 if geom == FAN else 180.0, nrows=1,
                    ncols=ncols, pixel_v=1.0, pixel_u=pixel_u, nx=nx, ny=ny, nz=1, voxel_xy=1.0, voxel_z=1.0, start_deg=11.0,
                    shift_u=0.3, center_x=0.7, center_y=-1.1).replace(**fan).replace(**kw)


SCANS = [scan(FAN, 1, 1, 1, 1), scan(FAN, 9, 7, 63, 3), scan(FAN, 64, 8, 64, 8), scan(FAN, 65, 71, 65, 17), scan(FAN, 130, 33, 129, 40),
         scan(FAN, 200, 200, 300, 50, pixel_u=1.9), scan(FAN, 40, 40, 200, 9, pixel_u=0.55), scan(FAN, 48, 48, 96, 12, pixel_u=3.9),
         scan(FAN, 140, 150, 96, 3, pixel_u=3.7),       # many waves, wide runs of voxels: the workgroup's LDS limits the split
         scan(PARALLEL, 1, 5, 2, 2), scan(PARALLEL, 64, 64, 96, 90, pixel_u=1.0), scan(PARALLEL, 17, 66, 64, 5, pixel_u=0.4),
         scan(PARALLEL, 90, 50, 70, 31, pixel_u=2.2), scan(PARALLEL, 30, 31, 40, 6, voxel_z=0.6, pixel_v=0.9, shift_v=0.4)]


def rel(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("cfg", SCANS, ids=lambda c: c.name)
@pytest.mark.parametrize("batch", [1, 3, 21])
def test_flat_kernels_match_oracle(oracle_mod, cfg, batch):
    import torch
    from paper_2307_05801_amd import Geometry, binding as B
    geo = Geometry(cfg)
    assert "A=general(flat" in geo.describe() and "AT=general(flat" in geo.describe(), geo.describe()
    print(f"[gpu] {cfg.name} batch={batch}: {geo.describe()}", flush=True)
    x, y = uniform_volume(cfg, 3, batch=batch), uniform_sinogram(cfg, 4, batch=batch)
    ax = geo.project(torch.from_numpy(x).cuda()).cpu().numpy()
    aty = geo.backproject(torch.from_numpy(y).cuda()).cpu().numpy()
    for b in {0, batch // 2, batch - 1}:
        assert rel(ax[b], oracle_mod.project(cfg, x[b])) <= TOL
        assert rel(aty[b], oracle_mod.backproject(cfg, y[b])) <= TOL
    # an item's sums do not depend on how many others it shares a launch with
    for b in {0, batch // 2, batch - 1}:
        one = geo.project(torch.from_numpy(x[b:b + 1]).cuda()).cpu().numpy(), geo.backproject(torch.from_numpy(y[b:b + 1]).cuda()).cpu().numpy()
        assert np.array_equal(one[0][0], ax[b]) and np.array_equal(one[1][0], aty[b])
    # nor on the copy: the fixed-scratch entry point reads the slices as they lie
    fixed = torch.full((batch,) + geo.sino_shape, float("nan"), device="cuda")
    xt = torch.from_numpy(x).cuda()
    B.leap_project_static_scratch(geo.handle, xt.data_ptr(), fixed.data_ptr(), batch, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert np.array_equal(fixed.cpu().numpy(), ax)
    geo.close()


def test_other_items_and_voxels_beside_a_beam_do_not_reach_it():
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(SCANS[3])
    x = torch.rand((5,) + geo.vol_shape, device="cuda")
    y = torch.rand((5,) + geo.sino_shape, device="cuda")
    ax, aty = geo.project(x), geo.backproject(y)
    xb, yb = x.clone(), y.clone()
    xb[1, 0, 40, 30] = float("nan")
    yb[3, 9, 0, 20] = float("inf")
    axb, atyb = geo.project(xb), geo.backproject(yb)
    # the rays through the voxel (and no others) are NaN, the voxels of the ray infinite
    w = torch.zeros_like(x[:1])
    w[0, 0, 40, 30] = 1.0
    hit = geo.project(w)[0] > 0
    assert torch.equal(axb[1].isnan(), hit) and torch.equal(axb[[0, 2, 3, 4]], ax[[0, 2, 3, 4]])
    r = torch.zeros_like(y[:1])
    r[0, 9, 0, 20] = 1.0
    hit = geo.backproject(r)[0] > 0
    assert torch.equal(~atyb[3].isfinite(), hit) and torch.equal(atyb[[0, 1, 2, 4]], aty[[0, 1, 2, 4]])
    geo.close()


def test_captured_calls_and_two_streams():
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(SCANS[4])
    x = torch.rand((9,) + geo.vol_shape, device="cuda")
    ref, out = geo.project(x), torch.empty((9,) + geo.sino_shape, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        geo.project(x, out=out)
    side = torch.cuda.Stream()
    for _ in range(3):
        x.uniform_()
        graph.replay()
        got = out.clone()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            other = geo.project(x)
        ref = geo.project(x)
        torch.cuda.synchronize()
        assert torch.equal(other, ref) and torch.equal(got, ref)
    geo.close()


@pytest.mark.parametrize("cfg", [scan(FAN, 131, 120, 129, 840), scan(FAN, 120, 131, 300, 520, pixel_u=0.9), scan(PARALLEL, 90, 50, 70, 400)], ids=lambda c: c.name)
def test_slices_turned_for_beams_along_x(oracle_mod, cfg):
    """Enough views that a batch is copied with its rows along y as well; an item alone reads the slice as it lies."""
    test_flat_kernels_match_oracle(oracle_mod, cfg, 5)
    test_flat_kernels_match_oracle(oracle_mod, cfg, 10)


@pytest.mark.parametrize("cfg", [scan(kind, 61, 67, nviews, 170) for kind in (PARALLEL, FAN) for nviews in (170, 171)], ids=lambda c: f"{c.name}-{c.nviews}")
def test_tiles_of_a_view_rounded_up_to_an_odd_number(oracle_mod, cfg):
    """More than two tiles of 64 columns, on either side of the number of workgroups from which they are rounded up, and a batch of three."""
    test_flat_kernels_match_oracle(oracle_mod, cfg, 3)


@pytest.mark.parametrize("cfg", [scan(kind, 40, 41, 60, nviews) for kind in (PARALLEL, FAN) for nviews in (64, 65)], ids=lambda c: c.name)
@pytest.mark.parametrize("batch", [5, 16, 23])
def test_groups_of_four_items_where_eight_leave_units_idle(oracle_mod, cfg, batch):
    """On either side of the number of workgroups, whole and ragged groups, and the rest of a batch that the scratch holds no more of."""
    test_flat_kernels_match_oracle(oracle_mod, cfg, batch)


@pytest.mark.parametrize("nx,ny", [(64, 64), (65, 64), (121, 61), (128, 64), (129, 64)])
@pytest.mark.parametrize("geom,nviews", [(PARALLEL, 64), (FAN, 63), (FAN, 64), (FAN, 131)])
def test_few_tiles_take_several_views_at_a_time(oracle_mod, geom, nx, ny, nviews):
    """Numbers of 8 x 8 tiles and of views on either side of the rule, in launches of one, two and three groups of items: the same bits."""
    cfg = scan(geom, nx, ny, 130, nviews, pixel_u=2.3 if geom == FAN else 1.3)
    test_flat_kernels_match_oracle(oracle_mod, cfg, 10)
    test_flat_kernels_match_oracle(oracle_mod, cfg, 21)
