"""Forward projection of few bundles, whose layers the waves of a workgroup share, and of short detectors on the column-wise kernels.

Layers shared by fewer blocks than waves, whole and slab by slab, against the oracle; a batch bit for bit what its items give alone;
scans of under 32 rows captured in a graph, and on the fixed scratch array, as from the general kernels that they ran on before."""
import pytest

from synthetic import CTConfig, perturbed_poses, uniform_volume
from synthetic.configs import CONE, CONE_CURVED, PARALLEL
from tests.test_gpu_parity import TOL, rel_l2

pytestmark = pytest.mark.gpu


def scan(geom, nrows, nviews=6, **kw):
    par = dict(sod=0.0, sdd=0.0) if geom == PARALLEL else dict(sod=150.0, sdd=225.0)
    base = dict(nviews=nviews, arc_deg=360.0, nrows=nrows, ncols=43, pixel_v=1.5, pixel_u=1.6, nx=41, ny=37, nz=max(8, nrows), voxel_xy=1.0,
                voxel_z=1.0, start_deg=3.0, shift_u=0.3, shift_v=-0.2)
    return CTConfig("parts", geom, **{**base, **par, **kw})


CASES = {"cone": (scan(CONE, 33), "sf"), "cone_8_rows": (scan(CONE, 8), "sf"), "cone_one_block": (scan(CONE, 40, nx=5, ny=7), "sf"),
         "cone_300_rows": (scan(CONE, 300, nviews=2), "sf"), "cone_520_rows": (scan(CONE, 520, nviews=2, nx=12, ny=13), "sf"),
         "curved": (scan(CONE_CURVED, 31), "sf"), "curved_200_rows": (scan(CONE_CURVED, 200, nviews=2), "sf"),
         "upright": (perturbed_poses(scan(CONE, 21), 5, shift_mm=4.0, upright=True), "sf"),
         "parallel": (scan(PARALLEL, 9), "sf"), "parallel_two_waves": (scan(PARALLEL, 70, nviews=160), "sf"),
         "parallel_500_rows": (scan(PARALLEL, 500, nviews=3), "sf"),
         "siddon_16_rows": (scan(CONE, 16), "siddon"), "siddon_parallel_22_rows": (scan(PARALLEL, 22), "siddon")}


@pytest.mark.parametrize("slab", ["", "slab=8"])
@pytest.mark.parametrize("name", list(CASES))
def test_shared_layers_and_short_detectors(oracle_mod, monkeypatch, name, slab):
    import torch
    from paper_2307_05801_amd import Geometry
    cfg, model = CASES[name]
    if slab:
        monkeypatch.setenv("LEAP_DEBUG", slab)
    geo = Geometry(cfg, model=model)
    print(f"[gpu] {name} {slab}: {geo.describe()}", flush=True)
    assert "A=columns" in geo.describe() and ("parts=" in geo.describe()) == (model == "sf"), geo.describe()
    assert ("parts=2" in geo.describe()) == (name == "parallel_two_waves"), geo.describe()
    x = uniform_volume(cfg, 5, batch=3)
    xt = torch.from_numpy(x).cuda()
    y = geo.project(xt)
    ref = (oracle_mod if model == "sf" else oracle_mod.siddon).project(cfg, x[1])
    assert rel_l2(y[1].cpu().numpy(), ref) <= TOL          # float sums of products whose positions are double: the parity tests' tolerance
    for b in range(3):
        assert torch.equal(y[b], geo.project(xt[b].contiguous())), b
    geo.close()


@pytest.mark.parametrize("geom", [CONE, CONE_CURVED, PARALLEL])
@pytest.mark.parametrize("nx", [4, 8, 9, 16, 17, 32, 33])
def test_slabs_of_fewer_blocks_than_waves(oracle_mod, monkeypatch, geom, nx):
    """Blocks are of 4 to 16 layers.  Waves without one are left out: the oracle's results, and those of a wave per bundle where there is one block."""
    import torch
    from paper_2307_05801_amd import Geometry
    cfg = scan(geom, 36, nviews=4, nx=nx, ny=max(4, nx - 1))
    geo = Geometry(cfg)
    print(f"[gpu] {geo.describe()}", flush=True)
    assert "parts=4" in geo.describe(), geo.describe()
    x = uniform_volume(cfg, 5)[0]
    xt = torch.from_numpy(x).cuda()
    y = geo.project(xt)
    assert rel_l2(y.cpu().numpy(), oracle_mod.project(cfg, x)) <= TOL
    monkeypatch.setenv("LEAP_DEBUG", "parts=1")
    plain = Geometry(cfg)
    slots = int(plain.describe().split("nq=")[1].split(",")[0].split("/")[1])
    if nx <= 64 // slots:
        assert torch.equal(y, plain.project(xt))
    plain.close()
    geo.close()


@pytest.mark.parametrize("name", ["cone", "cone_8_rows", "parallel"])
def test_items_of_a_large_batch_keep_their_bits(name):
    """Seventeen volumes, longer than wide, of whose copies the scratch holds fewer than sixteen."""
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(CASES[name][0].replace(nx=60, ny=37))
    print(f"[gpu] {name}: {geo.describe()}", flush=True)
    assert "parts=" in geo.describe(), geo.describe()
    x = torch.rand((17,) + tuple(geo.vol_shape), device="cuda")
    y = geo.project(x)
    for b in range(17):
        assert torch.equal(y[b], geo.project(x[b].contiguous())), b
    geo.close()


@pytest.mark.parametrize("name", ["cone_8_rows", "curved", "upright", "parallel", "siddon_16_rows"])
def test_short_detectors_captured_and_on_the_fixed_array(monkeypatch, name):
    """Neither needs a scratch, whatever stream the handle was last used on: the general kernel's results, bit for bit."""
    import torch
    from paper_2307_05801_amd import Geometry, binding
    cfg, model = CASES[name]
    geo = Geometry(cfg, model=model)
    monkeypatch.setenv("LEAP_DEBUG", "general=1")
    plain = Geometry(cfg, model=model)
    x = torch.rand((2,) + geo.vol_shape, device="cuda")
    want, eager = plain.project(x), geo.project(x)
    assert rel_l2(eager.cpu().numpy(), want.cpu().numpy()) <= 1e-6        # the same sums in another order, TOL's tenth
    out = torch.empty_like(want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        geo.project(x, out)
    for _ in range(3):
        x.copy_(torch.rand_like(x))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, plain.project(x))
        out.zero_()
    binding.leap_project_static_scratch(geo.handle, x.data_ptr(), out.data_ptr(), 2, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(out, plain.project(x))
    plain.close()
    geo.close()


def test_taller_detectors_captured():
    """A graph of a scan that uses the handle's scratch, after eager calls on another stream: two branches of the capture take the scratch in turn,
    and eager calls on other streams than the graph's follow."""
    import torch
    from paper_2307_05801_amd import Geometry
    geo = Geometry(CASES["cone"][0])
    x, z = (torch.rand(geo.vol_shape, device="cuda") for _ in range(2))
    ref_x, ref_z = geo.project(x), geo.project(z)
    out_x, out_z = torch.empty_like(ref_x), torch.empty_like(ref_z)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            geo.project(z, out_z)
        geo.project(x, out_x)
        torch.cuda.current_stream().wait_stream(side)
    for _ in range(4):
        out_x.zero_(), out_z.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_x, ref_x) and torch.equal(out_z, ref_z)
        with torch.cuda.stream(side):
            beside = geo.project(z)
        here = geo.project(x)
        torch.cuda.synchronize()
        assert torch.equal(here, ref_x) and torch.equal(beside, ref_z)
    geo.close()
