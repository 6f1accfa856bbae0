"""Footprint back projection of a few tiles and many views: the views shared among workgroups, each with a volume of its own.

Against the oracle; views that the parts and their groups of threads do not divide evenly; two items per workgroup and an odd last one; calls on
two streams; a captured call, which needs no room and takes the views in one workgroup."""
import pytest

from synthetic import CTConfig, perturbed_poses, uniform_sinogram
from synthetic.configs import CONE, CONE_CURVED, PARALLEL
from tests.test_gpu_parity import TOL, rel_l2

pytestmark = pytest.mark.gpu


def scan(geom=CONE, nviews=203, **kw):
    par = dict(sod=0.0, sdd=0.0) if geom == PARALLEL else dict(sod=150.0, sdd=225.0)
    base = dict(nviews=nviews, arc_deg=360.0, nrows=40, ncols=60, pixel_v=1.5, pixel_u=1.6, nx=37, ny=35, nz=27, voxel_xy=1.0, voxel_z=1.0,
                start_deg=3.0, shift_u=0.3)
    return CTConfig("parts", geom, **{**base, **par, **kw})


CASES = {"mirror": scan(), "off_centre": scan(shift_v=0.3), "odd_middle": scan(nz=29, nviews=331), "taller": scan(pixel_v=1.1, nrows=60, shift_v=0.2),
         "wide_window": scan(pixel_u=0.8, ncols=110, shift_v=0.2), "curved": scan(CONE_CURVED, shift_v=-0.2),
         "upright": perturbed_poses(scan(shift_v=0.2), 5, shift_mm=4.0, upright=True), "parallel": scan(PARALLEL, pixel_u=1.0, pixel_v=1.0, nviews=500)}


@pytest.mark.parametrize("name", list(CASES))
def test_parts_match_oracle(oracle_mod, name):
    import torch
    from paper_2307_05801_amd import Geometry
    cfg = CASES[name]
    geo = Geometry(cfg)
    print(f"[gpu] {name}: {geo.describe()}", flush=True)
    assert "+parts(" in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 5, batch=3)
    yt = torch.from_numpy(y).cuda()
    one = [geo.backproject(yt[b].contiguous()) for b in range(3)]
    # float sums whose positions are double: the parity tests' tolerance
    assert rel_l2(one[1].cpu().numpy(), oracle_mod.backproject(cfg, y[1])) <= TOL
    three = geo.backproject(yt)
    for b in range(3):
        assert torch.equal(one[b], geo.backproject(yt[b].contiguous()))
        # a batch takes the same parts as long as they are a gain, else its sums come in another order (a few roundings)
        assert rel_l2(three[b].cpu().numpy(), one[b].cpu().numpy()) <= 1e-6
    geo.close()


def test_two_streams_and_a_captured_call():
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(CASES["off_centre"])
    y, z = (torch.rand(geo.sino_shape, device="cuda") for _ in range(2))
    ref_y, ref_z, out = geo.backproject(y), geo.backproject(z), torch.empty(geo.vol_shape, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        geo.backproject(y, out=out)
    side = torch.cuda.Stream()
    for _ in range(3):
        out.zero_()
        graph.replay()
        captured = out.clone()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            beside = geo.backproject(z)
        here = geo.backproject(y)
        torch.cuda.synchronize()
        assert torch.equal(here, ref_y) and torch.equal(beside, ref_z)
        assert rel_l2(captured.cpu().numpy(), ref_y.cpu().numpy()) <= 1e-6
    geo.close()


@pytest.mark.parametrize("model,forward", [("sf", False), ("siddon", False), ("sf", True), ("siddon", True)])
def test_threads_on_their_per_thread_streams(model, forward):
    """hipStreamPerThread (the handle 2) is a stream of each thread's own: calls of two threads on one geometry share its memory in turn."""
    import threading
    import torch
    from paper_2307_05801_amd import Geometry, binding
    geo = Geometry(CASES["off_centre"].replace(nrows=24) if forward else CASES["off_centre"], model=model)
    print(f"[gpu] {model}: {geo.describe()}", flush=True)
    assert ("A=columns" if forward else "+parts(") in geo.describe(), geo.describe()
    run, operator = (binding.leap_project, geo.project) if forward else (binding.leap_backproject, geo.backproject)
    shape = geo.vol_shape if forward else geo.sino_shape
    src = [torch.rand(shape, device="cuda") for _ in range(2)]
    ref = [operator(s) for s in src]
    out = [[torch.empty_like(ref[0]) for _ in range(20)] for _ in range(2)]
    torch.cuda.synchronize()
    errors = []

    def work(n):
        try:
            for o in out[n]:
                run(geo.handle, src[n].data_ptr(), o.data_ptr(), 1, 2)
            torch.cuda.ExternalStream(2, device="cuda:0").synchronize()      # (the stream goes with its thread)
        except Exception as e:
            errors.append(e)

    threads = [threading.Thread(target=work, args=(n,)) for n in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    assert all(torch.equal(o, ref[n]) for n in range(2) for o in out[n])
    geo.close()


@pytest.mark.parametrize("model,forward", [("sf", False), ("siddon", False), ("sf", True), ("siddon", True)])
def test_six_streams_and_batches_beside_them(model, forward):
    """Single volumes on more streams than the memory has slots, and batches that take it whole between them."""
    import torch
    from paper_2307_05801_amd import Geometry
    cfg = CASES["off_centre"]
    geo = Geometry(cfg.replace(nrows=24) if forward else cfg, model=model)
    print(f"[gpu] {model}: {geo.describe()}", flush=True)
    assert ("A=columns" if forward else "+parts(") in geo.describe(), geo.describe()
    operator, shape = (geo.project, geo.vol_shape) if forward else (geo.backproject, geo.sino_shape)
    src = [torch.rand(shape, device="cuda") for _ in range(6)]
    many = torch.rand((12,) + tuple(shape), device="cuda")
    ref, ref_many = [operator(s) for s in src], operator(many)
    torch.cuda.synchronize()
    streams, got, got_many = [torch.cuda.Stream() for _ in src], [[] for _ in src], []
    for turn in range(8):
        for n, s in enumerate(streams):
            with torch.cuda.stream(s):
                got[n].append(operator(src[n]))
                if (turn + n) % 5 == 0:
                    got_many.append(operator(many))
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref[n]) for n in range(6) for o in got[n])
    assert got_many and all(torch.equal(o, ref_many) for o in got_many)
    geo.close()


SIDDON = {"cone": scan(shift_v=0.3), "parallel": scan(PARALLEL, pixel_u=1.0, pixel_v=1.0, nviews=500, shift_v=0.27), "curved": scan(CONE_CURVED, shift_v=-0.2),
          "upright": perturbed_poses(scan(shift_v=0.2), 5, shift_mm=4.0, upright=True),
          "tilted": perturbed_poses(scan(shift_v=0.2), 5, shift_mm=4.0, tilt_rad=0.05),
          "tilted_wide": perturbed_poses(scan(shift_v=0.2, pixel_u=0.9, ncols=100), 5, shift_mm=4.0, tilt_rad=0.05),
          "tilted_wide_tall": perturbed_poses(scan(shift_v=0.2, pixel_u=0.9, ncols=100, pixel_v=0.8, nrows=70), 5, shift_mm=4.0, tilt_rad=0.05)}


@pytest.mark.parametrize("name", list(SIDDON))
def test_siddon_parts_match_oracle(oracle_mod, name):
    import torch
    from paper_2307_05801_amd import Geometry
    cfg = SIDDON[name]
    geo = Geometry(cfg, model="siddon")
    print(f"[gpu] {name}: {geo.describe()}", flush=True)
    assert "+parts(" in geo.describe(), geo.describe()
    y = uniform_sinogram(cfg, 5, batch=3)
    yt = torch.from_numpy(y).cuda()
    one, three = geo.backproject(yt[1].contiguous()), geo.backproject(yt)
    assert rel_l2(one.cpu().numpy(), oracle_mod.siddon.backproject(cfg, y[1])) <= TOL
    assert rel_l2(three[1].cpu().numpy(), one.cpu().numpy()) <= 1e-6
    assert torch.equal(one, geo.backproject(yt[1].contiguous()))
    geo.close()


# name: scan, model, batch of which the room holds some items at a time (what each launch of theirs takes: test_host_logic.py)
ROUNDS = {"cone": (scan(nviews=301, nx=80, ny=95, nz=65, nrows=65, ncols=95, pixel_v=1.5, pixel_u=1.2, shift_v=0.3, sod=345.0, sdd=517.5), "sf", 7),
          "parallel": (scan(PARALLEL, nviews=180, nx=101, ny=105, nz=64, nrows=64, ncols=105, pixel_v=1.5, pixel_u=1.2, shift_v=0.3), "sf", 7),
          "siddon_cone": (scan(nviews=408, nx=43, ny=37, nz=11, nrows=11, ncols=43, shift_v=0.3, sod=189.0, sdd=283.5), "siddon", 21),
          "siddon_tilted": (perturbed_poses(scan(nviews=479, nx=12, ny=28, nz=14, nrows=14, ncols=28, shift_v=0.3), 5, shift_mm=3.0, tilt_rad=0.05), "siddon", 21)}


@pytest.mark.parametrize("name", list(ROUNDS))
def test_batches_that_take_the_room_several_times(oracle_mod, name):
    """Every item the bits it has by itself (a batch that takes the views as one volume does); the first and the last against the oracle."""
    import torch
    from paper_2307_05801_amd import Geometry
    cfg, model, batch = ROUNDS[name]
    geo = Geometry(cfg, model=model)
    print(f"[gpu] {name}: {geo.describe()}", flush=True)
    y = uniform_sinogram(cfg, 5, batch=batch)
    yt = torch.from_numpy(y).cuda()
    got = geo.backproject(yt)
    for b in range(batch):
        assert torch.equal(got[b], geo.backproject(yt[b].contiguous())), b
    for b in (0, batch - 1):
        assert rel_l2(got[b].cpu().numpy(), (oracle_mod if model == "sf" else oracle_mod.siddon).backproject(cfg, y[b])) <= TOL
    geo.close()
