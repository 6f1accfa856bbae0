"""Host logic of the HIP library, exercised on the CPU (no GPU): the real geometry module (validation, table
building, kernel selection and its static limits) linked against stubs of the HIP runtime, the general kernel bodies
stepped thread by thread, the window arithmetic of the tiled back projection, and the arithmetic of the column-wise
forward kernel.  tests/host/host_harness.cpp holds the C++ side."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_2307_05801_amd import binding as B
from synthetic import (CTConfig, config, modular_from, perturbed_poses, reduced, standard_volume, uniform_sinogram,
                       uniform_volume)
from synthetic.configs import CONE, CONE_CURVED, FAN, PARALLEL

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "host", "host_harness.cpp")
LIB = os.path.join(HERE, "host", "libhost_harness.so")
TOL = 1e-5


@pytest.fixture(scope="module")
def host():
    deps = [SRC, os.path.join(ROOT, "paper_2307_05801_amd", "csrc")]
    newest = max(os.path.getmtime(os.path.join(d, f)) if os.path.isdir(d) else os.path.getmtime(d)
                 for d in deps for f in (os.listdir(d) if os.path.isdir(d) else [""]))
    import fcntl
    with open(LIB + ".lock", "w") as lock:          # several pytest-xdist workers may arrive here together
        fcntl.flock(lock, fcntl.LOCK_EX)
        if not os.path.exists(LIB) or os.path.getmtime(LIB) < newest:
            tmp = f"{LIB}.{os.getpid()}.tmp"
            cmd = ["g++", "-O2", "-fopenmp", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                   "-I/opt/rocm/include", "-o", tmp, SRC,
                   os.path.join(ROOT, "paper_2307_05801_amd", "csrc", "leap_geometry.cpp"),
                   os.path.join(ROOT, "paper_2307_05801_amd", "csrc", "leap_host.cpp")]
            subprocess.run(cmd, check=True, capture_output=True)
            os.replace(tmp, LIB)
    lib = C.CDLL(LIB)
    B.declare(lib, solvers=False)
    lib.host_check_backproject_windows.argtypes = [C.c_void_p, C.POINTER(C.c_int64)]
    lib.host_project_columns.restype = C.c_long
    lib.host_project_columns.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p]
    lib.host_curved_column_deviation.argtypes = [C.c_void_p, C.POINTER(C.c_double)]
    lib.host_sd_project_columns.restype = C.c_long
    lib.host_sd_project_columns.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p]
    lib.host_mf_backproject_tiled.restype = C.c_long
    lib.host_mf_backproject_tiled.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.POINTER(C.c_int64)]
    lib.host_mf_project_tiles.restype = C.c_long
    lib.host_mf_project_tiles.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p]
    lib.host_project_rows.restype = lib.host_flat.restype = C.c_long
    lib.host_project_rows.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p]
    lib.host_flat.argtypes = [C.c_void_p] * 5 + [C.POINTER(C.c_int64)]
    lib.host_sd_project_pairs.restype = C.c_long
    lib.host_sd_project_pairs.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p]
    lib.host_sd_backproject_tiled.restype = C.c_long
    lib.host_sd_backproject_tiled.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.POINTER(C.c_int64)]
    lib.host_md_backproject_tiled.restype = C.c_long
    lib.host_md_backproject_tiled.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.POINTER(C.c_int64)]
    lib.host_md_project_columns.restype = C.c_long
    lib.host_md_project_columns.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int]
    return lib


def rel_l2(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


def handle(lib, cfg, model=B.LEAP_MODEL_SF):
    d, keep = B.desc_from_config(cfg, model)
    return B.leap_geometry_create(d, lib)


CASES = {
    "c1": (1, lambda: config(1)),
    "c2_div8": (2, lambda: reduced(config(2), 8, nviews=20)),
    "c3_div8_ragged": (3, lambda: reduced(config(3), 8, nviews=24).replace(nx=67, ny=70, nz=45, nrows=61, ncols=77)),
    "c3_div8_offsets": (3, lambda: reduced(config(3), 8, nviews=9).replace(
        shift_u=1.3, shift_v=-2.7, center_x=6.0, center_y=-4.5, center_z=3.25, start_deg=7.0)),
    "c4_div4": (4, lambda: reduced(config(4), 4, nviews=10)),
    "c5_div16": (5, lambda: reduced(config(5), 16, nviews=18)),
    "curved_c3_div8": (3, lambda: reduced(config(3), 8, nviews=24).replace(
        geom=CONE_CURVED, nx=67, ny=70, nz=45, nrows=61, ncols=77, shift_u=0.6, shift_v=-1.2, center_x=3.0)),
    "curved_wide_fan": (3, lambda: CTConfig("curved_wide", CONE_CURVED, nviews=16, arc_deg=360.0, nrows=48, ncols=120,
                                            pixel_v=2.0, pixel_u=1.6, nx=64, ny=60, nz=40, voxel_xy=1.0, voxel_z=1.2,
                                            sod=110.0, sdd=170.0, shift_u=-0.8, shift_v=0.3, center_y=1.5, start_deg=4.0)),
    # rows up to 1.9, 2.4 and 2.9 voxels tall: a pair of adjacent rows overlaps up to 5, 6 and 7 voxels
    "tall_rows_5": (3, lambda: reduced(config(3), 8, nviews=12).replace(pixel_v=8.0, nrows=56, voxel_z=3.4, nz=70, shift_v=0.3)),
    "tall_rows_6": (3, lambda: reduced(config(3), 8, nviews=12).replace(pixel_v=10.2, nrows=44, voxel_z=3.4, nz=70, center_z=2.0)),
    "tall_rows_7": (3, lambda: reduced(config(3), 8, nviews=12).replace(pixel_v=12.3, nrows=36, voxel_z=3.4, nz=70, shift_v=-0.4)),
    # rows under half a voxel tall: a pair stays within 2 voxels
    "short_rows_2": (3, lambda: reduced(config(3), 8, nviews=12).replace(pixel_v=2.3, nrows=200, voxel_z=4.0, nz=64)),
    # the source barely clears the volume's bounding circle (27.6 mm) and nx, ny are no multiples of the tile edge: the
    # padding voxels of the edge tiles reach past the source plane, where the window functions must stay defined
    "source_grazing_ragged_volume": (3, lambda: CTConfig("grazing", CONE, nviews=11, arc_deg=360.0, nrows=40, ncols=150,
                                                         pixel_v=1.5, pixel_u=1.5, nx=37, ny=41, nz=12, voxel_xy=1.0,
                                                         voxel_z=1.0, sod=28.5, sdd=60.0, shift_u=0.4, start_deg=2.0)),
    "fan": (3, lambda: CTConfig("fan", FAN, nviews=20, arc_deg=360.0, nrows=1, ncols=90, pixel_v=1.0, pixel_u=2.0,
                                nx=70, ny=64, nz=1, voxel_xy=1.0, voxel_z=1.0, sod=300.0, sdd=500.0, shift_u=0.8)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_general_kernel_bodies_match_oracle_on_cpu(host, oracle_mod, name):
    number, make = CASES[name]
    cfg = make()
    x = standard_volume(number, cfg) if cfg.nz > 1 or number == 1 else uniform_volume(cfg, 5)[0]
    y = uniform_sinogram(cfg, 50 + number)[0]
    h = handle(host, cfg)
    ax = np.zeros(cfg.sino_shape, np.float32)
    aty = np.zeros(cfg.vol_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ax.ctypes.data, 1, 0, host)
    B.leap_backproject(h, y.ctypes.data, aty.ctypes.data, 1, 0, host)
    B.leap_geometry_destroy(h, host)
    assert rel_l2(ax, oracle_mod.project(cfg, x)) <= TOL
    assert rel_l2(aty, oracle_mod.backproject(cfg, y)) <= TOL
    lhs, rhs = float((ax.astype(np.float64) * y).sum()), float((aty.astype(np.float64) * x).sum())
    assert abs(lhs - rhs) <= TOL * abs(lhs)


SIDDON_CASES = dict(CASES)
SIDDON_CASES["steep_thin_slices"] = (3, lambda: CTConfig(
    "steep", CONE, nviews=11, arc_deg=360.0, nrows=40, ncols=36, pixel_v=2.9, pixel_u=1.4, nx=30, ny=28, nz=60,
    voxel_xy=1.0, voxel_z=0.21, sod=40.0, sdd=62.0, shift_u=0.3, shift_v=-0.4, center_x=0.7, center_z=-0.3,
    start_deg=3.0))
SIDDON_CASES["parallel_3d"] = (3, lambda: CTConfig(
    "par3", PARALLEL, nviews=13, arc_deg=180.0, nrows=40, ncols=50, pixel_v=0.9, pixel_u=0.8, nx=40, ny=36, nz=21,
    voxel_xy=1.0, voxel_z=1.1, sod=0.0, sdd=0.0, shift_u=0.3, shift_v=-0.4, center_y=0.7, center_z=-0.3,
    start_deg=1.0))


@pytest.mark.parametrize("name", list(SIDDON_CASES))
def test_siddon_kernel_bodies_match_oracle_on_cpu(host, oracle_mod, name):
    number, make = SIDDON_CASES[name]
    cfg = make()
    # A thin ray that runs inside a voxel face plane (central column at an axis-aligned view) is a discontinuity of
    # the Siddon model: which side it falls on depends on the last bit of sin(pi).  Keep the pixel centres off them.
    cfg = cfg.replace(shift_u=cfg.shift_u + 0.123)
    x = standard_volume(number, cfg) if cfg.nz > 1 or number == 1 else uniform_volume(cfg, 5)[0]
    y = uniform_sinogram(cfg, 50 + number)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    ax = np.zeros(cfg.sino_shape, np.float32)
    aty = np.zeros(cfg.vol_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ax.ctypes.data, 1, 0, host)
    B.leap_backproject(h, y.ctypes.data, aty.ctypes.data, 1, 0, host)
    fast = np.zeros(cfg.sino_shape, np.float32)
    bad = host.host_sd_project_columns(h, x.ctypes.data, fast.ctypes.data)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    sd = oracle_mod.siddon
    assert ("A=columns" in desc) == (bad >= 0)
    assert ("A=columns" in desc) == (name not in ("c1", "fan", "steep_thin_slices")), desc
    if bad >= 0:
        assert bad == 0, desc
        assert rel_l2(fast, sd.project(cfg, x)) <= TOL, desc
    assert rel_l2(ax, sd.project(cfg, x)) <= TOL
    assert rel_l2(aty, sd.backproject(cfg, y)) <= TOL
    lhs, rhs = float((ax.astype(np.float64) * y).sum()), float((aty.astype(np.float64) * x).sum())
    assert abs(lhs - rhs) <= TOL * abs(lhs)


@pytest.mark.parametrize("name", ["c2_div8", "c3_div8_ragged", "c3_div8_offsets", "c4_div4", "c5_div16", "curved_c3_div8",
                                  "curved_wide_fan", "tall_rows_5", "tall_rows_6", "tall_rows_7", "short_rows_2"])
def test_column_forward_arithmetic_matches_oracle_on_cpu(host, oracle_mod, name, monkeypatch):
    number, make = CASES[name]
    cfg = make()
    x = standard_volume(number, cfg)
    ref = oracle_mod.project(cfg, x)
    for cw in ("1", "2", "4"):
        monkeypatch.setenv("LEAP_DEBUG", "cw=" + cw)
        h = handle(host, cfg)
        out = np.zeros(cfg.sino_shape, np.float32)
        uncovered = host.host_project_columns(h, x.ctypes.data, out.ctypes.data)
        desc = B.leap_geometry_describe(h, host)
        B.leap_geometry_destroy(h, host)
        assert uncovered == 0, desc
        assert rel_l2(out, ref) <= TOL, desc
        if name.startswith("tall_rows_") or name.startswith("short_rows_"):
            assert "nkp=" + name.rsplit("_", 1)[1] in desc, desc


def scratch_bytes(desc):
    return int(desc.split("scratch=")[1].split()[0])


@pytest.mark.parametrize("number", [2, 3, 4, 5])
@pytest.mark.parametrize("model", [B.LEAP_MODEL_SF, B.LEAP_MODEL_SIDDON])
def test_forward_scratch_is_bounded(host, number, model):
    """The z-fastest copy the fast forward kernels read holds one slab of the volume at a time: an eighth of the volume
    (a quarter with Siddon weights) from 512 MiB volumes on, 128 MiB for smaller ones."""
    cfg = config(number)
    h = handle(host, cfg, model)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert "A=columns" in desc, desc
    volume_bytes = 4 * cfg.nx * cfg.ny * cfg.nz
    if volume_bytes >= 512 << 20:
        bound = volume_bytes // (8 if model == B.LEAP_MODEL_SF else 4)
    else:
        bound = 128 << 20
    assert 0 < scratch_bytes(desc) <= bound, desc


def test_scratch_override_and_general_kernels_need_none(host, monkeypatch):
    cfg = reduced(config(3), 4, nviews=8)
    monkeypatch.setenv("LEAP_DEBUG", "slab=16,scratch_mib=3")
    h = handle(host, cfg)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert "slab=16" in desc and scratch_bytes(desc) == 3 << 20, desc
    monkeypatch.setenv("LEAP_DEBUG", "general=1")
    h = handle(host, cfg)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert "A=general" in desc and scratch_bytes(desc) == 0, desc


@pytest.mark.parametrize("case,model,tokens", [
    (2, B.LEAP_MODEL_SF, ("A=columns(", "cw=4", "AT=tiled(nc=3,nv=2,zc=64")),
    (3, B.LEAP_MODEL_SF, ("A=columns(", "rg=4,cw=4", "AT=tiled(nc=3,nv=2,zc=64")),
    (4, B.LEAP_MODEL_SF, ("A=columns(", "rg=3,cw=4", "AT=tiled(nc=4,nv=3,zc=16")),
    (5, B.LEAP_MODEL_SF, ("A=columns(", "rg=4,cw=4", "AT=tiled(nc=3,nv=3,zc=64")),
    (3, B.LEAP_MODEL_SIDDON, ("A=columns(rg=8", "AT=tiled(nc=2,zc=32")),
])
def test_benchmark_cases_take_the_instances_the_measurements_name(host, case, model, tokens):
    """The kernel instances the measured figures belong to: a change of the selection rules that moves a benchmark case
    to another instance (or to the general kernels) shows up here, on the CPU."""
    h = handle(host, config(case), model)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    for token in tokens:
        assert token in desc, desc


def test_row_schemes_of_the_tiled_back_projection_follow_the_voxel_height(host):
    """The three-row instance of the tiled back projection runs schemes that need every voxel at most two detector rows
    tall: a bound on the height within a thousandth of two rows takes the four-row instance, and volumes of 128 layers
    and more keep 64 voxels per thread for footprints up to two rows tall when their window fits."""
    base = reduced(config(2), 4, nviews=8)                 # parallel beam: a voxel is voxel_z / pixel_v rows tall
    for voxel_z, nz, token in ((0.99, 40, "nv=2,"), (1.0, 40, "nv=2,"), (1.25, 40, "nv=3,"), (1.99, 40, "nv=3,"),
                               (1.9995, 40, "nv=4,"), (2.4, 40, "nv=4,"),
                               (1.0, 160, "nv=2,zc=64"), (1.2, 160, "nv=3,zc=64"), (1.9, 160, "nv=3,zc=16")):
        cfg = base.replace(voxel_z=voxel_z, pixel_v=1.0, nz=nz, nrows=int(voxel_z * nz) + 12)
        h = handle(host, cfg)
        desc = B.leap_geometry_describe(h, host)
        B.leap_geometry_destroy(h, host)
        assert "AT=tiled" in desc and token in desc, (voxel_z, nz, desc)


def window_report(host, cfg):
    h = handle(host, cfg)
    rep = (C.c_int64 * 8)()
    host.host_check_backproject_windows(h, rep)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    return list(rep), desc


@pytest.mark.parametrize("name", ["c2_div8", "c3_div8_ragged", "c3_div8_offsets", "c4_div4", "c5_div16", "curved_c3_div8",
                                  "curved_wide_fan"])
def test_tiled_backprojection_reads_stay_inside_the_staged_window(host, name):
    rep, desc = window_report(host, CASES[name][1]())
    assert rep[0] == 1, desc
    assert rep[7] == 0, (rep, desc)


def level_rows(name, geom, **kw):
    """Odd detectors over volumes of even height: the middle row's rays run along a z-face (v is 0 or a rounding error)."""
    par = dict(sod=0.0, sdd=0.0) if geom == PARALLEL else dict(sod=150.0, sdd=225.0)
    return CTConfig(name, geom, nviews=7, arc_deg=360.0, nrows=67, ncols=60, pixel_v=0.7, pixel_u=1.1, nx=30, ny=28, nz=24, voxel_xy=1.0,
                    voxel_z=1.0, shift_u=0.123, start_deg=3.0, **par).replace(**kw)


SIDDON_TILED_CASES = {
    "c3_ragged": lambda: CASES["c3_div8_ragged"][1](), "offsets": lambda: CASES["c3_div8_offsets"][1](),
    "curved": lambda: CASES["curved_c3_div8"][1](), "parallel_3d": lambda: SIDDON_CASES["parallel_3d"][1](),
    "apart": lambda: level_rows("apart", CONE, nrows=40, pixel_v=1.9, shift_v=0.31),
    "upright": lambda: perturbed_poses(level_rows("up", CONE, pixel_v=1.3, shift_v=0.2), 5, shift_mm=3.0, upright=True),
    "level_parallel": lambda: level_rows("level_parallel", PARALLEL),
    "level_parallel_exact": lambda: level_rows("level_parallel_exact", PARALLEL, pixel_v=0.75),
    "level_parallel_fine": lambda: level_rows("level_parallel_fine", PARALLEL, nrows=131, pixel_v=0.35),
    "level_parallel_short": lambda: level_rows("level_parallel_short", PARALLEL, nrows=45, pixel_v=0.9),
    "level_cone_fine": lambda: level_rows("level_cone_fine", CONE, pixel_v=0.85),
    "level_parallel_apart": lambda: level_rows("level_parallel_apart", PARALLEL, nrows=69, pixel_v=1.25, nz=60),
    "level_cone": lambda: level_rows("level_cone", CONE, pixel_v=0.75), "level_cone_inexact": lambda: level_rows("level_cone_inexact", CONE),
}


@pytest.mark.parametrize("shape", ["bp_split=-1", "bp_split=0", "bp_split=1"])
@pytest.mark.parametrize("name", list(SIDDON_TILED_CASES))
def test_tiled_siddon_back_projection_matches_oracle_on_cpu(host, oracle_mod, monkeypatch, name, shape):
    monkeypatch.setenv("LEAP_DEBUG", shape)             # no shared views, shared under either shape (where its windows fit)
    cfg = SIDDON_TILED_CASES[name]()
    cfg = cfg.replace(shift_u=cfg.shift_u + 0.123)      # no rays inside vertical voxel faces
    y = uniform_sinogram(cfg, 4)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    aty = np.zeros(cfg.vol_shape, np.float32)
    rep = (C.c_int64 * 4)()
    bad = host.host_sd_backproject_tiled(h, y.ctypes.data, aty.ctypes.data, rep)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert bad == 0, (bad, list(rep), desc)
    want = oracle_mod.siddon.backproject(cfg, y)
    assert rel_l2(aty, want) <= 1e-6, desc
    assert np.abs(aty - want).max() <= 1e-5 * np.abs(want).max()


# (those with more than 64 rows; the back projection's list holds shorter detectors too)
SIDDON_PAIR_CASES = {n: m for n, m in SIDDON_TILED_CASES.items() if n.startswith("level") and n != "level_parallel_short"}
SIDDON_PAIR_CASES.update(
    cone=lambda: level_rows("cone", CONE, shift_v=0.31), cone_apart=lambda: level_rows("cone_apart", CONE, nrows=70, pixel_v=2.1, shift_v=0.31),
    cone_either_side=lambda: level_rows("cone_either_side", CONE, nrows=70, pixel_v=1.5), rows_finer=lambda: level_rows("finer", CONE, nrows=140, pixel_v=0.4),
    curved=lambda: level_rows("curved", CONE_CURVED, shift_v=0.2, pixel_v=1.3),
    upright=lambda: perturbed_poses(level_rows("up", CONE, pixel_v=1.3, shift_v=0.2), 5, shift_mm=3.0, upright=True))


@pytest.mark.parametrize("name", list(SIDDON_PAIR_CASES))
def test_siddon_pairs_match_oracle_on_cpu(host, oracle_mod, name):
    cfg = SIDDON_PAIR_CASES[name]()
    cfg = cfg.replace(shift_u=cfg.shift_u + 0.123)      # no rays inside vertical voxel faces
    x = uniform_volume(cfg, 3)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    ax = np.zeros(cfg.sino_shape, np.float32)
    bad = host.host_sd_project_pairs(h, x.ctypes.data, ax.ctypes.data)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert bad == 0, (bad, desc)
    want = oracle_mod.siddon.project(cfg, x)
    assert rel_l2(ax, want) <= 1e-6, desc
    assert np.abs(ax - want).max() <= 1e-5 * np.abs(want).max()


def test_siddon_pairs_add_what_the_weights_say(host):
    """One slab's value from its in-plane cells a, b and the lower and upper axial cell of each: a weight of zero adds nothing
    however large its voxel (the same bits), an infinite voxel of positive weight gives infinity."""
    host.host_sd_pair_slab.restype = C.c_float
    host.host_sd_pair_slab.argtypes = [C.c_float] * 4 + [C.c_int, C.c_int, C.c_float, C.c_float]

    def weights(two, inc, f, low):                  # alo, aup, blo, bup
        if not two:
            return np.array([low, 1.0 - low, 0.0, 0.0])
        la = min(low, f) if inc else max(low - (1.0 - f), 0.0)
        return np.array([la, f - la, low - la, 1.0 - f - (low - la)])

    rng = np.random.default_rng(5)
    for trial in range(6000):
        two, inc = trial % 3 != 0, trial % 2 == 0
        f = float(np.float32(rng.choice([rng.uniform(0, 1), 1e-3, 0.999, 0.5]))) if two else 1.0
        low = float(np.float32(rng.choice([rng.uniform(0, 1), 0.0, 1.0])))
        w, x = weights(two, inc, f, low), rng.uniform(0.5, 2.0, 4).astype(np.float32)

        def slab(v):
            return host.host_sd_pair_slab(*(float(t) for t in v), two, inc, f, low)

        # weights good to 2^-24 each, four products and sums
        assert abs(slab(x) - w @ x) <= 8 * 2.0 ** -24 * np.abs(x).sum(), (two, inc, f, low, x)
        for c in range(4 if two else 2):
            y = x.copy()
            if low in (0.0, 1.0) and w[c] == 0.0:
                for big in (1e8, -3e38):
                    y[c] = big
                    assert slab(y) == slab(x), (two, inc, f, low, c, big)
            elif w[c] > 1e-4:
                y[c] = np.inf
                assert slab(y) == np.inf, (two, inc, f, low, c)
    for low in (0.25, 0.5):
        assert host.host_sd_pair_slab(np.inf, np.inf, 0.0, 0.0, 0, 1, 1.0, low) == np.inf


def test_flat_scans_beyond_one_launch_keep_the_general_kernels(host):
    """65535 views of 65537 columns are 1025 wavefronts per view, more than 2^32 threads."""
    def describe(ncols):
        cfg = CTConfig("long", PARALLEL, nviews=65535, arc_deg=180.0, nrows=1, ncols=ncols, pixel_v=1.0, pixel_u=1.0, nx=8, ny=8, nz=1,
                       voxel_xy=1.0, voxel_z=1.0)
        h = handle(host, cfg)
        desc = B.leap_geometry_describe(h, host)
        B.leap_geometry_destroy(h, host)
        return desc
    assert "flat" in describe(64)
    assert "flat" not in describe(65537)


def test_flat_launches_hold_what_the_selection_admits(host):
    """Fewer than 2^32 threads of 64 per view and tile, although an even number of tiles is rounded up to an odd one."""
    assert [host.host_flat_tiles(c, v) for c, v in ((128, 4000), (129, 100), (256, 128), (256, 129), (320, 200))] == [2, 3, 4, 5, 5]
    for tiles, nviews in ((671088, 100), (671087, 100), (671086, 100), (1024, 65535), (1022, 65535), (4, 65535)):
        assert tiles * nviews * 64 < 1 << 32
        assert host.host_flat_tiles(64 * tiles, nviews) * nviews * 64 < 1 << 32, (tiles, nviews)
    assert host.host_flat_tiles(64 * 671088, 100) == 671088 and host.host_flat_tiles(64 * 671086, 100) == 671087


def test_every_staged_sample_has_one_writer(host):
    """Two threads that write one LDS cell in different steps race, even where they mean to write the same value."""
    host.host_check_staging_roles.restype = C.c_long
    assert host.host_check_staging_roles() == 0


@pytest.mark.parametrize("name", ["curved_c3_div8", "curved_wide_fan"])
def test_curved_tile_relative_columns_agree_with_the_general_function(host, name):
    """The tiled back projection takes a voxel column's fan angle relative to its tile's centre and the corner angles
    from a short series.  Against the general function (double atan2, atanf) the column coordinate may move by the
    float roundings of the small angle (four of them: about 2.4e-7 x angle x pixels per radian, a few 1e-6 pixel on
    these cases), the knot offsets by less."""
    h = handle(host, CASES[name][1]())
    out = (C.c_double * 3)()
    assert host.host_curved_column_deviation(h, out) == 0
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert "AT=tiled" in desc, desc
    assert out[0] < 4e-6 and out[1] < 1e-6, list(out)
    assert out[2] < 0.08, list(out)


@pytest.mark.parametrize("ncols,pixel_u", [(200, 2.0), (33, 8.0), (31, 9.0)])
def test_curved_bundle_relative_columns_agree_with_the_general_function(host, ncols, pixel_u):
    """The column-wise forward projection takes a voxel column's fan angle relative to its bundle's middle ray, from fine pixels to
    ones so wide that the angles come near the polynomials' end.  Column coordinate: double throughout, relative error 7e-13 of a
    few pixels.  Knot offsets: float, both functions within a few roundings (6e-8) of up to 4 pixels, atanf's own 2 ulp among them."""
    cfg = CTConfig("curved_near", CONE_CURVED, nviews=7, arc_deg=360.0, nrows=40, ncols=ncols, pixel_v=2.5, pixel_u=pixel_u,
                   nx=40, ny=37, nz=16, voxel_xy=2.0, voxel_z=2.0, sod=90.0, sdd=180.0, shift_u=0.3)
    h = handle(host, cfg)
    out = (C.c_double * 5)()
    host.host_curved_bundle_deviation.argtypes = [C.c_void_p, C.POINTER(C.c_double)]
    assert host.host_curved_bundle_deviation(h, out) == 0
    B.leap_geometry_destroy(h, host)
    assert out[4] > 1000 and out[3] < 0.32, list(out)
    assert out[0] < 2e-11 and out[1] < 2e-6 and out[2] < 1e-14, list(out)


def test_curved_source_too_close_for_the_series(host):
    """Corner angles above 0.08 rad: the tiled curved kernel is not chosen."""
    cfg = CTConfig("curved_close", CONE_CURVED, nviews=8, arc_deg=360.0, nrows=40, ncols=64, pixel_v=2.5, pixel_u=2.5,
                   nx=16, ny=16, nz=16, voxel_xy=2.0, voxel_z=2.0, sod=28.0, sdd=60.0)
    h = handle(host, cfg)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert "AT=general" in desc, desc


def test_window_limits_at_full_benchmark_sizes(host):
    """Every tile and chunk of a spread of views of the 512^3 and 1024^3 cone-beam cases, and the batch case."""
    for cfg in (config(3).with_views(list(range(0, 720, 45))), config(5).with_views([0, 181, 542, 1260]), config(4)):
        rep, desc = window_report(host, cfg)
        assert rep[0] == 1 and rep[7] == 0, (rep, desc)


def test_kernel_selection(host):
    def desc(cfg):
        h = handle(host, cfg)
        s = B.leap_geometry_describe(h, host)
        B.leap_geometry_destroy(h, host)
        return s
    assert "A=columns" in desc(config(3)) and "AT=tiled" in desc(config(3))
    assert "A=general" in desc(CASES["fan"][1]()) and "AT=general" in desc(CASES["fan"][1]())
    assert "A=general" in desc(config(1))                                  # one detector row: nothing to tile
    coarse = reduced(config(3), 8, nviews=4).replace(pixel_u=37.0, pixel_v=29.0, nrows=14, ncols=12)
    assert "A=general" in desc(coarse)                                     # a row spans six voxels
    fine = reduced(config(3), 8, nviews=4).replace(pixel_u=1.7, pixel_v=1.9, nrows=300, ncols=280)
    assert "AT=general" in desc(fine)                                      # a voxel spans six pixels


@pytest.mark.parametrize("seed", range(24))
def test_random_geometries_on_cpu(host, oracle_mod, seed):
    """Whatever kernels a random scanner selects, their static limits hold and the arithmetic matches the oracle."""
    from random_geometries import random_config
    cfg = random_config(seed)
    x = uniform_volume(cfg, seed)[0]
    y = uniform_sinogram(cfg, seed)[0]
    h = handle(host, cfg)
    desc = B.leap_geometry_describe(h, host)
    rep = (C.c_int64 * 8)()
    host.host_check_backproject_windows(h, rep)
    assert rep[7] == 0, (list(rep), desc)
    ref = oracle_mod.project(cfg, x)
    out = np.zeros(cfg.sino_shape, np.float32)
    uncovered = host.host_project_columns(h, x.ctypes.data, out.ctypes.data)
    if uncovered >= 0:
        assert uncovered == 0, desc
        assert rel_l2(out, ref) <= TOL, desc
    ax = np.zeros(cfg.sino_shape, np.float32)
    aty = np.zeros(cfg.vol_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ax.ctypes.data, 1, 0, host)
    B.leap_backproject(h, y.ctypes.data, aty.ctypes.data, 1, 0, host)
    B.leap_geometry_destroy(h, host)
    assert rel_l2(ax, ref) <= TOL, desc
    assert rel_l2(aty, oracle_mod.backproject(cfg, y)) <= TOL, desc


MODULAR_CASES = {
    "cone_as_modular": lambda: modular_from(reduced(config(3), 16, nviews=10).replace(shift_u=0.123)),
    "tilted_modules": lambda: perturbed_poses(reduced(config(3), 16, nviews=9).replace(nx=29, ny=35, nz=22, nrows=27, ncols=31),
                                              3, shift_mm=20.0, tilt_rad=0.25),
    "looking_down": lambda: CTConfig("down", 4, nviews=2, arc_deg=360.0, nrows=20, ncols=24, pixel_v=1.5, pixel_u=1.4,
                                     nx=18, ny=16, nz=12, voxel_xy=1.0, voxel_z=1.3, shift_u=0.2, shift_v=-0.3,
                                     poses=((0.3, -0.2, 40.0, 0.0, 0.0, -30.0, 1.0, 0.0, 0.0, 0.0, 1.0, 0.0),
                                            (6.0, 2.0, 38.0, -2.0, 1.0, -28.0, 0.8, 0.6, 0.0, -0.6, 0.8, 0.0))),
}


@pytest.mark.parametrize("name", list(MODULAR_CASES))
def test_modular_siddon_bodies_match_oracle_on_cpu(host, oracle_mod, name):
    cfg = MODULAR_CASES[name]()
    x = uniform_volume(cfg, 5)[0]
    y = uniform_sinogram(cfg, 6)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    ax = np.zeros(cfg.sino_shape, np.float32)
    aty = np.zeros(cfg.vol_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ax.ctypes.data, 1, 0, host)
    B.leap_backproject(h, y.ctypes.data, aty.ctypes.data, 1, 0, host)
    B.leap_geometry_destroy(h, host)
    sd = oracle_mod.siddon
    assert rel_l2(ax, sd.project(cfg, x)) <= TOL
    assert rel_l2(aty, sd.backproject(cfg, y)) <= TOL
    if name == "cone_as_modular":
        cone = reduced(config(3), 16, nviews=10).replace(shift_u=0.123)
        assert rel_l2(ax, sd.project(cone, x)) <= TOL


TILTED_FOOTPRINT_CASES = {
    "tilted_modules": MODULAR_CASES["tilted_modules"],
    "tilted_tall_voxels": lambda: perturbed_poses(
        reduced(config(3), 16, nviews=7).replace(nx=23, ny=19, nz=9, voxel_z=3.1, nrows=33, ncols=29), 8, shift_mm=15.0,
        tilt_rad=0.35),
    "looking_down_obliquely": lambda: CTConfig(
        "down", 4, nviews=2, arc_deg=360.0, nrows=20, ncols=24, pixel_v=1.5, pixel_u=1.4, nx=18, ny=16, nz=12,
        voxel_xy=1.0, voxel_z=1.3, shift_u=0.2, shift_v=-0.3,
        poses=((30.0, -4.0, 40.0, -22.0, 3.0, -30.0, 0.0, 1.0, 0.0, 0.8, 0.0, -0.6),
               (6.0, 34.0, 38.0, -2.0, -25.0, -28.0, 0.8, 0.6, 0.0, -0.36, 0.48, -0.8))),
    "mixed_upright_and_tilted": lambda: _mixed_scan(),
}


def _mixed_scan():
    base = reduced(config(3), 16, nviews=8).replace(nx=21, ny=26, nz=17, nrows=25, ncols=30)
    t = perturbed_poses(base, 5, shift_mm=10.0, tilt_rad=0.2)
    u = perturbed_poses(base, 5, shift_mm=10.0, tilt_rad=0.2, upright=True)
    return t.replace(poses=tuple(t.poses[a] if a % 2 else u.poses[a] for a in range(t.nviews)))


@pytest.mark.parametrize("name", list(TILTED_FOOTPRINT_CASES))
def test_tilted_footprint_bodies_match_oracle_on_cpu(host, oracle_mod, name):
    """The one-thread-per-ray / per-voxel bodies of the footprint model on tilted modules, stepped on the CPU."""
    cfg = TILTED_FOOTPRINT_CASES[name]()
    x = uniform_volume(cfg, 5)[0]
    y = uniform_sinogram(cfg, 6)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SF)
    desc = B.leap_geometry_describe(h, host)
    assert "tilted modules" in desc and "A=general" in desc and "AT=general" in desc, desc
    ax = np.zeros(cfg.sino_shape, np.float32)
    aty = np.zeros(cfg.vol_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ax.ctypes.data, 1, 0, host)
    B.leap_backproject(h, y.ctypes.data, aty.ctypes.data, 1, 0, host)
    B.leap_geometry_destroy(h, host)
    ref_a, ref_t = oracle_mod.project(cfg, x), oracle_mod.backproject(cfg, y)
    assert np.abs(ref_a).max() > 0 and np.abs(ref_t).max() > 0
    assert rel_l2(ax, ref_a) <= 1e-6 and rel_l2(aty, ref_t) <= 1e-6
    assert np.abs(ax - ref_a).max() <= 2e-6 * np.abs(ref_a).max()
    assert np.abs(aty - ref_t).max() <= 2e-6 * np.abs(ref_t).max()


@pytest.mark.parametrize("shift", [dict(shift_u=3e6), dict(shift_v=-3e6), dict(shift_u=-1e9), dict(shift_u=1e12)])
@pytest.mark.parametrize("name", ["c3_div8_ragged", "curved_c3_div8"])
def test_tiled_back_projections_far_beside_the_detector(host, name, shift):
    cfg = CASES[name][1]()
    cfg = cfg.replace(geom=CONE if name != "curved_c3_div8" or "shift_u" in shift else CONE_CURVED, **{k: v + 0.3 for k, v in shift.items()})
    rep, desc = window_report(host, cfg)
    assert rep[7] == 0, (list(rep), desc)
    y = uniform_sinogram(cfg, 4)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    aty, rep4 = np.zeros(cfg.vol_shape, np.float32), (C.c_int64 * 4)()
    assert host.host_sd_backproject_tiled(h, y.ctypes.data, aty.ctypes.data, rep4) in (0, -1), list(rep4)
    B.leap_geometry_destroy(h, host)
    tilted = perturbed_poses(level_rows("tilted", CONE, nx=40, ny=40), 3, shift_mm=2.0, tilt_rad=0.1).replace(**{k: v + 0.3 for k, v in shift.items()})
    y = uniform_sinogram(tilted, 4)[0]
    h = handle(host, tilted, B.LEAP_MODEL_SIDDON)
    aty, rep3 = np.zeros(tilted.vol_shape, np.float32), (C.c_int64 * 3)()
    assert host.host_md_backproject_tiled(h, y.ctypes.data, aty.ctypes.data, rep3) in (0, -1), list(rep3)
    B.leap_geometry_destroy(h, host)


TILED_FOOTPRINT_CASES = {
    "ragged": dict(nx=17, ny=20, nz=11, nrows=70, ncols=37, pixel=1.5), "wide_angles": dict(nx=20, ny=15, nz=9, nrows=40, ncols=50, pixel=1.5, tilt=0.5),
    "fine_pixels": dict(nx=9, ny=8, nz=10, nrows=90, ncols=60, pixel=0.45), "coarse_pixels": dict(nx=20, ny=18, nz=10, nrows=20, ncols=24, pixel=3.7),
    "far_columns": dict(nx=9, ny=8, nz=10, nrows=20, ncols=24, pixel=1.5, shift_u=100000.25)}


def tiled_footprint_scan(nx, ny, nz, nrows, ncols, pixel, tilt=0.1, **kw):
    base = CTConfig("tiled", CONE, nviews=6, arc_deg=360.0, nrows=nrows, ncols=ncols, pixel_v=pixel, pixel_u=pixel, nx=nx, ny=ny, nz=nz,
                    voxel_xy=1.0, voxel_z=1.1, sod=160.0, sdd=240.0, shift_v=-0.3, center_x=1.0, center_y=-2.0, center_z=0.5, start_deg=3.0)
    return perturbed_poses(base, 3, shift_mm=4.0, tilt_rad=tilt).replace(**kw)


@pytest.mark.parametrize("name", list(TILED_FOOTPRINT_CASES))
def test_tiled_tilted_footprints_match_oracle_on_cpu(host, oracle_mod, name):
    cfg = tiled_footprint_scan(**TILED_FOOTPRINT_CASES[name])
    x, y = uniform_volume(cfg, 3)[0], uniform_sinogram(cfg, 4)[0]
    h = handle(host, cfg)
    ax, aty, rep = np.zeros(cfg.sino_shape, np.float32), np.zeros(cfg.vol_shape, np.float32), (C.c_int64 * 2)()
    beside = host.host_mf_project_tiles(h, x.ctypes.data, ax.ctypes.data)
    bad = host.host_mf_backproject_tiled(h, y.ctypes.data, aty.ctypes.data, rep)
    B.leap_geometry_destroy(h, host)
    assert beside == 0 and bad == 0, (beside, list(rep))
    for got, want in ((ax, oracle_mod.project(cfg, x)), (aty, oracle_mod.backproject(cfg, y))):
        assert np.linalg.norm(got - want) <= 6e-8 * np.linalg.norm(want) + 1e-12


@pytest.mark.parametrize("shift_u", [0.0, 3e5, 3e6, 3e7, 1e9, 1e12])
def test_tiled_tilted_footprints_far_beside_the_detector(host, shift_u):
    """Columns far from the detector's own: a float holds a window's bounds to a fraction of a pixel only so far out."""
    cfg = tiled_footprint_scan(nx=40, ny=40, nz=16, nrows=40, ncols=50, pixel=1.37, shift_u=shift_u + 0.3)
    y = uniform_sinogram(cfg, 4)[0]
    h = handle(host, cfg)
    aty, rep = np.zeros(cfg.vol_shape, np.float32), (C.c_int64 * 2)()
    bad = host.host_mf_backproject_tiled(h, y.ctypes.data, aty.ctypes.data, rep)
    B.leap_geometry_destroy(h, host)
    assert bad == 0 or bad == -1, (bad, list(rep))
    assert bad == 0 or shift_u > 1e5


def test_tilted_scans_without_footprints_are_refused(host):
    """A source beside the volume with the module on the far side of only part of it, and a module below a source that
    looks straight down: LEAP_BAD_GEOMETRY with a message, as the oracle refuses them."""
    base = dict(nviews=1, arc_deg=360.0, nrows=20, ncols=24, pixel_v=1.5, pixel_u=1.4, nx=18, ny=16, nz=12, voxel_xy=1.0,
                voxel_z=1.3)
    grazing = (10.5, 0.0, 0.0, -30.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.6, 0.0, 0.8)       # the plane's normal tilts: corners behind
    below = (0.3, -0.2, 40.0, 0.0, 0.0, -30.0, 1.0, 0.0, 0.0, 0.0, 1.0, 0.0)
    for pose in (grazing, below):
        cfg = CTConfig("bad", 4, poses=(pose,), **base)
        with pytest.raises(B.LeapError) as err:
            handle(host, cfg, B.LEAP_MODEL_SF)
        assert err.value.status == B.LEAP_BAD_GEOMETRY and "no footprints" in str(err.value)
    # a source 0.2 mm in front of the volume's face: the nearest voxels' footprints span hundreds of pixels
    roll = np.sqrt(1 - 0.01)
    close = (9.2, 0.0, 0.0, -300.0, 0.0, 0.0, 0.0, roll, -0.1, 0.0, 0.1, roll)        # rolled about its normal (the x axis)
    with pytest.raises(B.LeapError) as err:
        handle(host, CTConfig("close", 4, poses=(close,), **base), B.LEAP_MODEL_SF)
    assert err.value.status == B.LEAP_UNSUPPORTED and "64 pixels" in str(err.value)


UPRIGHT_CASES = {
    "cone_as_modular": lambda: modular_from(reduced(config(3), 16, nviews=10).replace(shift_u=0.3, shift_v=-0.4)),
    "shifted_upright_modules": lambda: perturbed_poses(
        reduced(config(3), 16, nviews=9).replace(nx=29, ny=35, nz=22, nrows=41, ncols=31), 3, shift_mm=25.0, tilt_rad=0.3,
        upright=True),
    "wobbly_orbit": lambda: perturbed_poses(reduced(config(5), 32, nviews=12), 11, shift_mm=10.0, tilt_rad=0.1, upright=True),
}


@pytest.mark.parametrize("name", list(UPRIGHT_CASES))
def test_modular_footprint_bodies_match_oracle_on_cpu(host, oracle_mod, name):
    cfg = UPRIGHT_CASES[name]()
    x = uniform_volume(cfg, 5)[0]
    y = uniform_sinogram(cfg, 6)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SF)
    ax = np.zeros(cfg.sino_shape, np.float32)
    aty = np.zeros(cfg.vol_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ax.ctypes.data, 1, 0, host)
    B.leap_backproject(h, y.ctypes.data, aty.ctypes.data, 1, 0, host)
    # the fast kernels' host-side re-enactments on the per-view parameter blocks
    rep = (C.c_int64 * 8)()
    host.host_check_backproject_windows(h, rep)
    fast = np.zeros(cfg.sino_shape, np.float32)
    uncovered = host.host_project_columns(h, x.ctypes.data, fast.ctypes.data)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    ref = oracle_mod.project(cfg, x)
    assert rel_l2(ax, ref) <= TOL
    assert rel_l2(aty, oracle_mod.backproject(cfg, y)) <= TOL
    assert "AT=tiled" in desc and rep[0] == 1 and rep[7] == 0, (list(rep), desc)
    if name != "wobbly_orbit":          # that one has 32 detector rows at most: below the column kernel's minimum
        assert "A=columns" in desc, desc
    if uncovered >= 0:
        assert uncovered == 0, desc
        assert rel_l2(fast, ref) <= TOL, desc


@pytest.mark.parametrize("name", list(UPRIGHT_CASES))
def test_upright_modular_siddon_uses_the_ray_table(host, oracle_mod, name):
    """Upright modules get the Siddon model's per-column ray table, built on each view's own parameter block: the
    column kernel's host re-enactment must reproduce the oracle and stay inside the scratch volume."""
    cfg = UPRIGHT_CASES[name]()
    x = standard_volume(3, cfg)
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    fast = np.zeros(cfg.sino_shape, np.float32)
    bad = host.host_sd_project_columns(h, x.ctypes.data, fast.ctypes.data)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert "upright" in desc and "AT=tiled" in desc, desc
    assert "A=columns" in desc and bad == 0, (bad, desc)
    assert rel_l2(fast, oracle_mod.siddon.project(cfg, x)) <= TOL, desc


def test_modular_argument_checks(host):
    cfg = MODULAR_CASES["looking_down"]()
    d, keep = B.desc_from_config(cfg, B.LEAP_MODEL_SF)
    hnd = C.c_void_p()
    assert host.leap_geometry_create(C.byref(d), C.byref(hnd)) == B.LEAP_BAD_GEOMETRY     # a pixel's ray runs along z: no footprint
    d, keep = B.desc_from_config(cfg, B.LEAP_MODEL_SIDDON)
    d.poses = C.POINTER(C.c_double)()
    assert host.leap_geometry_create(C.byref(d), C.byref(hnd)) == B.LEAP_INVALID_ARG
    skew = cfg.replace(poses=((0.3, -0.2, 40.0, 0.0, 0.0, -30.0, 1.0, 0.0, 0.0, 0.1, 1.0, 0.0),) * 2)
    d, keep = B.desc_from_config(skew, B.LEAP_MODEL_SIDDON)
    assert host.leap_geometry_create(C.byref(d), C.byref(hnd)) == B.LEAP_INVALID_ARG
    inside = cfg.replace(poses=((0.3, -0.2, 1.0, 0.0, 0.0, -30.0, 1.0, 0.0, 0.0, 0.0, 1.0, 0.0),) * 2)
    d, keep = B.desc_from_config(inside, B.LEAP_MODEL_SIDDON)
    assert host.leap_geometry_create(C.byref(d), C.byref(hnd)) == B.LEAP_BAD_GEOMETRY


OUT_OF_MEMORY = """
import ctypes as C, sys
sys.path[:0] = [{root!r}, {here!r}]
import test_host_logic as T
from paper_2307_05801_amd import binding as B
lib = C.CDLL(T.LIB)
B.declare(lib, solvers=False)
lib.host_fail_allocation.restype, lib.host_fail_allocation.argtypes = C.c_long, [C.c_long]
failures = 0
for cfg, model in T.memory_scans():
    d, keep = B.desc_from_config(cfg, model)
    h = C.c_void_p()
    lib.host_fail_allocation(-1)
    assert lib.leap_geometry_create(C.byref(d), C.byref(h)) == 0
    lib.leap_geometry_destroy(h)
    total = lib.host_fail_allocation(-1)
    for n in list(range(min(total, 60))) + list(range(60, total, max(1, total // 60))):
        lib.host_fail_allocation(n)
        status = lib.leap_geometry_create(C.byref(d), C.byref(h))
        if status != 0:
            assert not h.value and lib.leap_last_error(), (cfg.name, n)
            failures += 1
        else:
            lib.leap_geometry_destroy(h)
    lib.host_fail_allocation(-1)
    print(cfg.name, total, failures, flush=True)
assert failures > 30
print("done")
"""


def memory_scans():
    cone = level_rows("cone", CONE, nviews=72)
    return [(cone, 0), (cone, 1), (cone.replace(geom=CONE_CURVED), 0), (level_rows("par", PARALLEL, nviews=72), 0),
            (perturbed_poses(cone, 5, shift_mm=3.0, upright=True), 0), (perturbed_poses(cone, 5, shift_mm=3.0, tilt_rad=0.1), 0),
            (perturbed_poses(cone, 5, shift_mm=3.0, tilt_rad=0.1), 1)]


def test_creation_that_runs_out_of_host_memory_reports_it(host):
    """Every allocation of leap_geometry_create fails once, those of its worker threads among them: a status, no abort."""
    import sys
    res = subprocess.run([sys.executable, "-c", OUT_OF_MEMORY.format(root=ROOT, here=HERE)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "done" in res.stdout, (res.returncode, res.stdout[-500:], res.stderr[-1500:])


def test_host_memory_pipeline_rotates_buffers_and_chunks_correctly(host, monkeypatch):
    """leap_project_host / leap_backproject_host against the device-pointer calls, with every asynchronous HIP call
    of the pipeline carried out at once (the harness' stubs): 5 items through the two-deep buffer rotation, staging
    buffers of 4 KiB so that every array takes many chunks with a ragged last one, both directions on one handle."""
    monkeypatch.setenv("LEAP_DEBUG", "stage_kib=4")
    cfg = reduced(config(3), 32, nviews=5).replace(nx=19, ny=17, nz=11, nrows=13, ncols=23)
    batch = 5
    x = np.stack([uniform_volume(cfg, 20 + b)[0] for b in range(batch)])
    y = np.stack([uniform_sinogram(cfg, 40 + b)[0] for b in range(batch)])
    h = handle(host, cfg)
    ax_ref = np.zeros((batch,) + cfg.sino_shape, np.float32)
    aty_ref = np.zeros((batch,) + cfg.vol_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ax_ref.ctypes.data, batch, 0, host)
    B.leap_backproject(h, y.ctypes.data, aty_ref.ctypes.data, batch, 0, host)
    ax = np.full_like(ax_ref, np.nan)
    aty = np.full_like(aty_ref, np.nan)
    B.leap_project_host(h, x.ctypes.data, ax.ctypes.data, batch, host)
    B.leap_backproject_host(h, y.ctypes.data, aty.ctypes.data, batch, host)      # arrays of the other sizes on the same handle
    one = np.full(cfg.sino_shape, np.nan, np.float32)
    B.leap_project_host(h, x[3].ctypes.data, one.ctypes.data, 1, host)
    with pytest.raises(B.LeapError):
        B.leap_project_host(h, x.ctypes.data, x.ctypes.data, 1, host)
    with pytest.raises(B.LeapError):
        B.leap_project_host(h, x.ctypes.data, ax.ctypes.data, 0, host)
    B.leap_geometry_destroy(h, host)
    assert np.array_equal(ax, ax_ref) and np.array_equal(aty, aty_ref) and np.array_equal(one, ax_ref[3])


TILTED_SIDDON_FAST_CASES = {
    "tilted_modules": lambda: perturbed_poses(reduced(config(3), 16, nviews=9).replace(nx=29, ny=35, nz=22, nrows=43, ncols=31),
                                              3, shift_mm=20.0, tilt_rad=0.25),
    "wobbly_tilted_orbit": lambda: perturbed_poses(reduced(config(5), 32, nviews=12), 11, shift_mm=10.0, tilt_rad=0.1),
    "tall_voxels": lambda: perturbed_poses(
        reduced(config(3), 16, nviews=7).replace(nx=23, ny=19, nz=9, voxel_z=3.1, nrows=33, ncols=29), 8, shift_mm=15.0,
        tilt_rad=0.35),
}


@pytest.mark.parametrize("name", list(TILTED_SIDDON_FAST_CASES))
@pytest.mark.parametrize("width", [4, 1000])
def test_tilted_siddon_slab_kernel_matches_oracle_on_cpu(host, oracle_mod, name, width):
    """The per-lane slab walk of the tilted-module Siddon forward kernel, re-enacted slab by slab with the kernel's own
    functions (narrow slabs of 4 layers, and the whole volume at once)."""
    cfg = TILTED_SIDDON_FAST_CASES[name]()
    x = uniform_volume(cfg, 5)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    desc = B.leap_geometry_describe(h, host)
    out = np.zeros(cfg.sino_shape, np.float32)
    bad = host.host_md_project_columns(h, x.ctypes.data, out.ctypes.data, width)
    B.leap_geometry_destroy(h, host)
    assert "A=columns" in desc and "tilted modules" in desc and bad == 0, (bad, desc)
    ref = oracle_mod.siddon.project(cfg, x)
    assert rel_l2(out, ref) <= TOL, desc
    assert np.abs(out - ref).max() <= 2e-5 * np.abs(ref).max()


def test_steep_or_close_tilted_scans_keep_the_general_siddon_kernels(host):
    """Rays that rise by more than a cell per slab (modules seen obliquely from above), and a source within a voxel of the
    volume's box: the per-lane slab kernel is not chosen."""
    for cfg in (TILTED_FOOTPRINT_CASES["looking_down_obliquely"]().replace(nrows=40), MODULAR_CASES["looking_down"]().replace(nrows=40)):
        h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
        desc = B.leap_geometry_describe(h, host)
        B.leap_geometry_destroy(h, host)
        assert "A=general" in desc, desc
    base = reduced(config(3), 16, nviews=4).replace(nx=24, ny=24, nz=16, nrows=40, ncols=30)
    near = perturbed_poses(base, 2, shift_mm=1.0, tilt_rad=0.1)
    half = 0.5 * base.nx * base.voxel_xy
    poses = [list(p) for p in near.poses]
    poses[1][0:3] = [half + 0.5 * base.voxel_xy, 0.0, 0.0]           # half a voxel outside the +x face
    poses[1][3:6] = [-300.0, 0.0, 0.0]
    h = handle(host, near.replace(poses=tuple(tuple(p) for p in poses)), B.LEAP_MODEL_SIDDON)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert "A=general" in desc, desc


def far_scanner(**kw):
    """A cone-beam scanner whose source keeps more than a hundred voxels from the volume (what the tiled back projection
    on tilted modules asks for), small enough for the CPU."""
    base = dict(name="far", geom=2, nviews=9, arc_deg=360.0, nrows=48, ncols=56, pixel_v=1.5, pixel_u=1.5, nx=37, ny=41,
                nz=29, voxel_xy=1.0, voxel_z=1.0, sod=160.0, sdd=240.0, shift_u=0.3, shift_v=-0.4, center_x=1.0,
                center_y=-2.0, center_z=0.5, start_deg=3.0)
    base.update(kw)
    return CTConfig(**base)


TILTED_SIDDON_TILED_CASES = {
    "small_tilts": lambda: perturbed_poses(far_scanner(), 3, shift_mm=4.0, tilt_rad=0.05),
    "rolled_modules": lambda: perturbed_poses(far_scanner(nviews=7), 5, shift_mm=6.0, tilt_rad=0.3),
    "tall_voxels": lambda: perturbed_poses(far_scanner(nz=19, voxel_z=1.7, nviews=8), 8, shift_mm=5.0, tilt_rad=0.15),
}


@pytest.mark.parametrize("shape", ["bp_split=-1", "bp_split=0", "bp_split=1"])
@pytest.mark.parametrize("name", list(TILTED_SIDDON_TILED_CASES))
def test_tilted_siddon_tiled_back_projection_matches_oracle_on_cpu(host, oracle_mod, monkeypatch, name, shape):
    """The tiled back projection on tilted modules re-enacted tile by tile with the kernel's own functions: every staged
    window fits, every read stays inside it, every slot inside the sums, and the result is the oracle's."""
    monkeypatch.setenv("LEAP_DEBUG", shape)
    cfg = TILTED_SIDDON_TILED_CASES[name]()
    y = uniform_sinogram(cfg, 6)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    desc = B.leap_geometry_describe(h, host)
    out = np.full(cfg.vol_shape, np.nan, np.float32)
    rep = (C.c_int64 * 4)()
    bad = host.host_md_backproject_tiled(h, y.ctypes.data, out.ctypes.data, rep)
    B.leap_geometry_destroy(h, host)
    assert "AT=tiled" in desc and bad == 0, (bad, list(rep), desc)
    ref = oracle_mod.siddon.backproject(cfg, y)
    assert rel_l2(out, ref) <= TOL, desc
    assert np.abs(out - ref).max() <= 2e-5 * np.abs(ref).max()


def test_host_memory_pipeline_with_threaded_staging_copies(host, monkeypatch):
    """Staging buffers of 1 MiB: every chunk's copy to or from pinned memory is shared out among the helper threads, and
    arrays of 2.4 and 1.6 MB take a ragged last chunk."""
    monkeypatch.setenv("LEAP_DEBUG", "stage_kib=1024")
    cfg = reduced(config(3), 8, nviews=6).replace(nx=96, ny=96, nz=64, nrows=96, ncols=112)
    batch = 3
    x = np.stack([uniform_volume(cfg, 60 + b)[0] for b in range(batch)])
    h = handle(host, cfg)
    ref = np.zeros((batch,) + cfg.sino_shape, np.float32)
    B.leap_project(h, x.ctypes.data, ref.ctypes.data, batch, 0, host)
    ax = np.full_like(ref, np.nan)
    B.leap_project_host(h, x.ctypes.data, ax.ctypes.data, batch, host)
    back_ref = np.zeros((batch,) + cfg.vol_shape, np.float32)
    B.leap_backproject(h, ref.ctypes.data, back_ref.ctypes.data, batch, 0, host)
    back = np.full_like(back_ref, np.nan)
    B.leap_backproject_host(h, ref.ctypes.data, back.ctypes.data, batch, host)
    B.leap_geometry_destroy(h, host)
    assert np.array_equal(ax, ref) and np.array_equal(back, back_ref)


def test_large_scans_behind_a_source_plane_are_refused_for_the_siddon_model(host):
    """A module turned 60 degrees away from the line source - volume and rolled a little: the plane through the source
    parallel to the module cuts the volume, so the general back projection would test every pixel for the voxels behind
    it.  Tiny scans run that way (the oracle agrees); at 256^3 x 256^2 the handle is refused."""
    c, s_ = np.cos(np.pi / 3), np.sin(np.pi / 3)
    n = np.array([c, s_, 0.0])
    eu = np.array([-s_, c, 0.0]) * np.sqrt(1 - 0.01) + np.array([0.0, 0.0, -0.1])
    ev = np.cross(n, eu)
    S = np.array([200.0, 0.0, 0.0])
    pose = tuple(np.concatenate([S, S - 300.0 * n, eu / np.linalg.norm(eu), ev / np.linalg.norm(ev)]))
    big = CTConfig("cut", 4, nviews=4, arc_deg=360.0, nrows=256, ncols=256, pixel_v=1.0, pixel_u=1.0, nx=256, ny=256, nz=256,
                   voxel_xy=1.0, voxel_z=1.0, poses=(pose,) * 4)
    with pytest.raises(B.LeapError) as err:
        handle(host, big, B.LEAP_MODEL_SIDDON)
    assert err.value.status == B.LEAP_UNSUPPORTED and "behind the source's plane" in str(err.value)
    small = big.replace(nrows=24, ncols=24, nx=20, ny=20, nz=20, voxel_xy=12.8, voxel_z=12.8, pixel_u=10.0, pixel_v=10.0)
    h = handle(host, small, B.LEAP_MODEL_SIDDON)
    assert "AT=general" in B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)


@pytest.mark.parametrize("seed", range(16))
def test_flatness_decision_of_tilted_siddon_scans_matches_brute_force(host, seed):
    """The per-lane slab kernel is chosen iff no ray rises by more than 0.999 axial cells per slab along its faster in-plane
    axis.  The library decides that by clipping the detector's rectangle with four half-planes per view; here every pixel
    (and a 4 x finer grid between the pixel centres) is simply tried."""
    rng = np.random.default_rng([seed, 77])
    base = far_scanner(nviews=6, voxel_z=float(rng.uniform(0.5, 2.0)), nz=int(rng.integers(10, 40)))
    cfg = perturbed_poses(base, seed, shift_mm=float(rng.uniform(0, 30)), tilt_rad=float(rng.uniform(0.05, 1.3)))
    lift = float(rng.uniform(0.0, 260.0))            # sources raised above the volume: their rays dive
    cfg = cfg.replace(poses=tuple(tuple(np.asarray(p) + np.array([0, 0, lift * (a % 2)] + [0] * 9)) for a, p in enumerate(cfg.poses)))
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    fast = "A=columns" in B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    kappa = cfg.voxel_xy / cfg.voxel_z
    u = (np.linspace(0, cfg.ncols - 1, 4 * cfg.ncols - 3) - (cfg.ncols - 1) / 2 + cfg.shift_u) * cfg.pixel_u
    v = (np.linspace(0, cfg.nrows - 1, 4 * cfg.nrows - 3) - (cfg.nrows - 1) / 2 + cfg.shift_v) * cfg.pixel_v
    uu, vv = np.meshgrid(u, v)
    worst = 0.0
    for p in cfg.poses:
        p = np.asarray(p)
        D = (p[3:6] - p[0:3]) + uu[..., None] * p[6:9] + vv[..., None] * p[9:12]
        with np.errstate(divide="ignore"):
            worst = max(worst, float((kappa * np.abs(D[..., 2]) / np.maximum(np.abs(D[..., 0]), np.abs(D[..., 1]))).max()))
    if worst > 1.0:
        assert not fast, worst
    elif worst < 0.99:
        assert fast, worst          # (these scanners keep every source far more than a voxel from the volume)


@pytest.mark.parametrize("seed", range(8))
def test_tilted_siddon_kernels_on_random_scans_match_oracle_on_cpu(host, oracle_mod, seed):
    """Random tilts (up to 0.5 rad about every axis), shifts, voxel aspect ratios and sizes: wherever the library picks the
    per-lane kernels, their re-enactments stay inside their buffers and agree with the oracle."""
    from random_geometries import random_tilted_scan
    cfg = random_tilted_scan(seed)
    x, y = uniform_volume(cfg, 5)[0], uniform_sinogram(cfg, 6)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    desc = B.leap_geometry_describe(h, host)
    sd = oracle_mod.siddon
    checked = 0
    if "A=columns" in desc:
        out = np.zeros(cfg.sino_shape, np.float32)
        assert host.host_md_project_columns(h, x.ctypes.data, out.ctypes.data, 8) == 0, desc
        assert rel_l2(out, sd.project(cfg, x)) <= TOL, desc
        checked += 1
    if "AT=tiled" in desc:
        out = np.full(cfg.vol_shape, np.nan, np.float32)
        rep = (C.c_int64 * 4)()
        assert host.host_md_backproject_tiled(h, y.ctypes.data, out.ctypes.data, rep) == 0, (list(rep), desc)
        ref = sd.backproject(cfg, y)
        assert rel_l2(out, ref) <= TOL and np.abs(out - ref).max() <= 2e-5 * np.abs(ref).max(), desc
        checked += 1
    B.leap_geometry_destroy(h, host)
    assert checked >= 1, desc


@pytest.mark.parametrize("pixel_u,pixel_v,tiles", [(0.45, 0.45, True), (0.25, 0.25, True), (0.2, 0.2, False), (0.12, 1.5, True),
                                                   (1.5, 0.12, False), (0.5, 0.15, True), (0.1, 0.5, False)])
def test_forward_tiles_of_tilted_footprints_are_left_where_voxels_cover_many_pixels(host, pixel_u, pixel_v, tiles):
    base = CTConfig("fine", CONE, nviews=8, arc_deg=360.0, nrows=40, ncols=40, pixel_v=pixel_v, pixel_u=pixel_u, nx=32, ny=32, nz=32,
                    voxel_xy=1.0, voxel_z=1.0, sod=80.0, sdd=120.0, start_deg=3.0)
    h = handle(host, perturbed_poses(base, 3, shift_mm=2.0, tilt_rad=0.05))
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert ("A=general(tiles)" in desc) == tiles, desc


@pytest.mark.parametrize("nrows,pixel_v,nz,kw", [(32, 1.9, 57, {}), (65, 0.9, 57, {}), (200, 0.31, 57, {}), (40, 2.9, 110, {}),
                                                 (90, 1.3, 57, dict(shift_v=60.0)), (64, 1.0, 64, dict(shift_v=0.0, center_z=0.0))])
def test_projection_by_rows_matches_oracle_on_cpu(host, oracle_mod, nrows, pixel_v, nz, kw):
    cfg = CTConfig("rows", PARALLEL, nviews=7, arc_deg=180.0, nrows=nrows, ncols=75, pixel_v=pixel_v, pixel_u=1.1, nx=41, ny=50, nz=nz,
                   voxel_xy=1.0, voxel_z=1.0, shift_u=0.3, shift_v=-0.4, center_x=1.0, center_y=-2.0, center_z=0.5, start_deg=3.0).replace(**kw)
    x = uniform_volume(cfg, 3)[0]
    h = handle(host, cfg)
    ax = np.zeros(cfg.sino_shape, np.float32)
    bad = host.host_project_rows(h, x.ctypes.data, ax.ctypes.data)
    B.leap_geometry_destroy(h, host)
    assert bad == 0
    assert np.linalg.norm(ax - oracle_mod.project(cfg, x)) <= 1e-6 * np.linalg.norm(oracle_mod.project(cfg, x))


@pytest.mark.parametrize("geom,nx,ny,ncols,pixel_u,kw", [
    (FAN, 65, 71, 65, 1.3, {}), (FAN, 9, 7, 63, 1.3, {}), (FAN, 100, 90, 200, 1.4, dict(sod=150.0, sdd=260.0)), (FAN, 40, 40, 200, 0.55, {}),
    (FAN, 48, 48, 96, 3.9, {}), (PARALLEL, 17, 66, 64, 0.4, {}), (PARALLEL, 90, 50, 70, 2.2, {}), (PARALLEL, 30, 31, 40, 1.1, dict(voxel_z=0.6, shift_v=0.4))])
def test_flat_kernels_match_oracle_on_cpu(host, oracle_mod, geom, nx, ny, ncols, pixel_u, kw):
    fan = dict(sod=400.0, sdd=700.0) if geom == FAN else {}
    cfg = CTConfig("flat", geom, nviews=23, arc_deg=360.0, nrows=1, ncols=ncols, pixel_v=1.0, pixel_u=pixel_u, nx=nx, ny=ny, nz=1, voxel_xy=1.0,
                   voxel_z=1.0, start_deg=11.0, shift_u=0.3, center_x=0.7, center_y=-1.1).replace(**fan).replace(**kw)
    x, y = uniform_volume(cfg, 3)[0], uniform_sinogram(cfg, 4)[0]
    h = handle(host, cfg)
    ax, aty, rep = np.zeros(cfg.sino_shape, np.float32), np.zeros(cfg.vol_shape, np.float32), (C.c_int64 * 2)()
    bad = host.host_flat(h, x.ctypes.data, ax.ctypes.data, y.ctypes.data, aty.ctypes.data, rep)
    B.leap_geometry_destroy(h, host)
    assert bad == 0, (bad, list(rep))
    for got, want in ((ax, oracle_mod.project(cfg, x)), (aty, oracle_mod.backproject(cfg, y))):
        assert np.linalg.norm(got - want) <= 2e-6 * np.linalg.norm(want)


def test_waves_of_a_flat_workgroup_take_every_slab_once(host):
    for nwaves in (1, 2, 4, 8, 16):
        assert not any(host.host_check_flat_shares(n, nwaves) for n in list(range(1, 300)) + [16383, 65536, 268435455])


@pytest.mark.parametrize("nx,ny,nz,wide", [(157, 167, 140, False), (176, 176, 160, False), (192, 192, 160, True), (211, 187, 149, True),
                                           (192, 192, 133, False)])
def test_wide_windows_need_enough_workgroups(host, nx, ny, nz, wide):
    """550, 605, 720 and 840 workgroups of 32 voxels per thread; 720 with a sixth of the layers as padding."""
    cfg = CTConfig("w", CONE, nviews=8, arc_deg=360.0, nrows=int(1.3 * nz), ncols=int(1.5 * nx), pixel_v=1.45, pixel_u=1.5, nx=nx, ny=ny, nz=nz,
                   voxel_xy=1.0, voxel_z=1.0, sod=2.2 * nx, sdd=3.08 * nx, start_deg=3.0)
    h = handle(host, cfg)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert ("zc=32,wide" in desc) == wide, desc


def scan_of(n, nviews, nrows, ncols, pixel_v=1.4, geom=CONE):
    return CTConfig("batch", geom, nviews=nviews, arc_deg=360.0, nrows=nrows, ncols=ncols, pixel_v=pixel_v, pixel_u=1.5, nx=n, ny=n, nz=n,
                    voxel_xy=1.0, voxel_z=1.0, sod=2.6 * n, sdd=3.9 * n, shift_u=0.3, shift_v=0.2)


@pytest.mark.parametrize("cfg,pairs", [
    # workgroups of one group of rows: views times column tiles of eight or sixteen
    (scan_of(64, 30, 70, 89), {2: 0, 3: 0, 4: 4, 5: 0, 8: 8, 16: 16}),       # 360 a volume
    (scan_of(64, 90, 70, 89), {2: 2, 3: 0, 4: 4, 5: 0, 8: 8}),               # 1080
    (scan_of(64, 180, 70, 89), {1: 0, 2: 2, 3: 2, 7: 6, 16: 16}),            # 2160
    # several groups of rows
    (scan_of(192, 40, 200, 268), {2: 0, 3: 0, 4: 4, 8: 8}),                  # two groups, 680
    (scan_of(192, 60, 264, 268), {2: 2, 3: 0, 4: 4, 5: 0, 8: 8}),            # three, 1020: one round of workgroups, two, four
    (scan_of(192, 250, 264, 268), {2: 2, 3: 2, 8: 8}),                       # 4250
    (config(4), {1: 0, 2: 0, 3: 0, 4: 4, 6: 6, 7: 0, 8: 8}),                 # 1440: a round and a half, three rounds
    # rows of 1.5 voxels and more: one group only, of two voxels and more: none (but on a cylinder)
    (scan_of(64, 180, 46, 89, pixel_v=2.2), {2: 2, 3: 2}),
    (scan_of(192, 180, 264, 268, pixel_v=2.2), {2: 0, 8: 0, 16: 0}),
    (scan_of(64, 720, 70, 89, pixel_v=3.4), {2: 0, 16: 0}),
    (scan_of(64, 180, 70, 89, pixel_v=3.4, geom=CONE_CURVED), {2: 2, 3: 2}),
])
def test_two_volumes_per_wave_need_waves_enough(host, cfg, pairs):
    """Batches whose pairs would leave the chip idle, and odd ones whose last item would, go one volume per wave."""
    h = handle(host, cfg)
    assert {items: host.host_forward_paired(C.c_void_p(h), items) for items in pairs} == pairs, B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)


@pytest.mark.parametrize("pixel_v,voxels", [(0.57, 2), (0.75, 3), (1.5, 4), (2.2, 5), (2.9, 7)])
def test_pairs_of_rows_read_no_more_voxels_than_they_overlap(host, pixel_v, voxels):
    """Rows of up to half a voxel, a voxel, a voxel and a half, two, three."""
    h = handle(host, scan_of(64, 8, 60, 89, pixel_v=pixel_v))
    assert host.host_voxels_of_pair(C.c_void_p(h)) == voxels, B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)


def small_scan(n, nviews, nz=None, shift_v=0.0, pixel=1.0, geom=PARALLEL):
    par = geom == PARALLEL
    nz = nz or n
    return CTConfig("small", geom, nviews=nviews, arc_deg=180.0, nrows=int(1.1 * nz / pixel), ncols=int(1.4 * n / pixel),
                    pixel_v=pixel if par else 1.5 * pixel, pixel_u=pixel if par else 1.5 * pixel, nx=n, ny=n, nz=nz, voxel_xy=1.0, voxel_z=1.0,
                    sod=0.0 if par else 2.6 * n, sdd=0.0 if par else 3.9 * n, shift_u=0.3, shift_v=shift_v)


# shapes: 0, 1, 2: 32, 16, 8 voxels per thread; what was measured fastest or within a few per cent of it
@pytest.mark.parametrize("cfg,shapes", [
    (small_scan(64, 60), {1: 2, 4: 2, 16: 0}),                          # mirror image
    (small_scan(64, 60, shift_v=0.2), {1: 2, 2: 2, 8: 2, 16: 0}),
    (small_scan(96, 60), {1: 2, 2: 2, 8: -1, 16: -1}),
    (small_scan(96, 8, shift_v=0.2), {1: 1, 2: 1, 16: -1}),
    (small_scan(64, 1), {1: -1, 16: -1}),                               # a single view: 12 us unsplit, up to 23 split
    (small_scan(100, 60, pixel=0.6), {1: 2, 2: 2, 16: -1}),             # wide windows
    (small_scan(224, 60, shift_v=0.2), {1: -1, 16: -1}),                # the chip is full
    (small_scan(96, 119, pixel=0.9, geom=CONE, shift_v=0.3), {1: 2, 16: -1}),
])
def test_views_are_shared_where_the_launch_leaves_the_chip_idle(host, cfg, shapes):
    """By the launch's workgroups, its items among them, and its views: a large batch of small volumes, or few views, are faster unsplit."""
    h = handle(host, cfg)
    got = {items: host.host_back_split_shape(C.c_void_p(h), items) for items in shapes}
    assert got == shapes, B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)


@pytest.mark.parametrize("cfg,pairs", [
    (small_scan(134, 60, nz=67, shift_v=0.2, pixel=1.4), {2: 0, 3: 0, 5: 0, 8: 4, 16: 8}),
    (small_scan(134, 8, nz=67, shift_v=0.2, pixel=1.4), {5: 0, 8: 4}),
    (small_scan(134, 1, nz=67, shift_v=0.2, pixel=1.4), {5: 0, 16: 0}),
    (small_scan(134, 60, nz=67, pixel=1.4), {1: 0, 16: 0}),             # mirror image: too few workgroups for two volumes in each
    (small_scan(256, 60), {1: 1, 3: 3}),                                # ... and enough
])
def test_two_items_per_workgroup_where_there_are_workgroups_enough(host, cfg, pairs):
    h = handle(host, cfg)
    assert {items: host.host_back_pairs(C.c_void_p(h), items) for items in pairs} == pairs, B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)


@pytest.mark.parametrize("pixel_u,shape", [(1.5, "zc=32,wide,window"), (1.1, "zc=16,window")])
def test_mirror_image_under_wide_windows(host, pixel_u, shape):
    """51 columns and 16 + 16 voxels where 42 columns do not hold the windows, 42 columns and 32 voxels of one volume where they do."""
    cfg = CTConfig("w", CONE, nviews=8, arc_deg=360.0, nrows=180, ncols=400, pixel_v=1.45, pixel_u=pixel_u, nx=224, ny=224, nz=160,
                   voxel_xy=1.0, voxel_z=1.0, sod=493.0, sdd=690.0, start_deg=3.0)
    h = handle(host, cfg)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert shape in desc and ("+mirror(zc=16,51x48)" in desc) == ("wide" not in desc), desc


# shapes: 0, 1: 16, 8 voxels per thread; tilted modules 8 voxels under 32, 64 columns
@pytest.mark.parametrize("cfg,shapes", [
    (small_scan(64, 60, shift_v=0.2), {1: 1, 4: 1, 16: -1}),
    (small_scan(96, 60, shift_v=0.2), {1: 0, 4: -1, 16: -1}),
    (small_scan(128, 8, shift_v=0.2), {1: 0, 16: -1}),
    (small_scan(64, 1, shift_v=0.2), {1: -1, 16: -1}),
    (small_scan(200, 60, shift_v=0.2), {1: -1, 16: -1}),
    ("tilted", {1: 0, 4: 0, 16: -1}),
])
def test_siddon_views_are_shared_where_the_launch_leaves_the_chip_idle(host, cfg, shapes):
    if cfg == "tilted":
        cfg = perturbed_poses(small_scan(64, 60, shift_v=0.2, pixel=1.3, geom=CONE).replace(nrows=54, ncols=68), 5, shift_mm=2.0, tilt_rad=0.05)
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    got = {items: host.host_siddon_split_shape(C.c_void_p(h), items) for items in shapes}
    assert got == shapes, B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)


@pytest.mark.parametrize("model,kind", [(B.LEAP_MODEL_SF, "curved"), (B.LEAP_MODEL_SIDDON, "tilted")])
def test_back_projections_left_to_the_general_kernel_are_described_as_such(host, model, kind):
    """The tables of the tiled kernels find no room on the device, or the source is too close for the cylinder's: nothing is left of the
    choices that go with those kernels."""
    cfg = small_scan(48, 8, geom=CONE_CURVED if kind == "curved" else CONE).replace(nrows=60, ncols=90)
    if kind == "tilted":
        cfg = perturbed_poses(small_scan(64, 8, shift_v=0.2, pixel=1.3, geom=CONE).replace(nrows=54, ncols=68), 5, shift_mm=2.0, tilt_rad=0.05)
    described = []
    for n in range(12):
        host.host_fail_device_allocation(C.c_long(n))
        try:
            h = handle(host, cfg, model)
        except B.LeapError:
            continue
        finally:
            host.host_fail_device_allocation(C.c_long(-1))
        described.append(B.leap_geometry_describe(h, host))
        B.leap_geometry_destroy(h, host)
    assert any("AT=tiled" in d and "+split" in d for d in described), described
    assert any("AT=general" in d for d in described), described
    assert not any("AT=general" in d and "+" in d.split("AT=")[1].split(" ")[0] for d in described), described
    close = CTConfig("curved_close", CONE_CURVED, nviews=8, arc_deg=360.0, nrows=40, ncols=64, pixel_v=2.5, pixel_u=2.5,
                     nx=16, ny=16, nz=16, voxel_xy=2.0, voxel_z=2.0, sod=28.0, sdd=60.0)
    h = handle(host, close)
    assert "AT=general " in B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)


@pytest.mark.parametrize("model", [B.LEAP_MODEL_SF, B.LEAP_MODEL_SIDDON])
@pytest.mark.parametrize("debug,tokens,absent", [
    ("bp_shape=1", ("tiled(",), ("+",)), ("bp_shape=3,bp_split=1", ("zc=16", "+split("), ("+mirror(", "+pairs(")),
    ("bp_split=-1,bp_pair=-1", ("tiled(",), ("+",)), ("bp_split=1", ("+split(",), ())])
def test_a_tile_shape_asked_for_is_the_one_that_runs(host, monkeypatch, model, debug, tokens, absent):
    """LEAP_DEBUG=bp_shape=N: no kernel of two volumes or of shared views in its place, unless one is named."""
    monkeypatch.setenv("LEAP_DEBUG", debug)
    h = handle(host, small_scan(64, 60, shift_v=0.0 if model == B.LEAP_MODEL_SF else 0.2), model)
    desc = B.leap_geometry_describe(h, host).split("AT=")[1].split(" scratch")[0]
    B.leap_geometry_destroy(h, host)
    assert all(t in desc for t in tokens) and not any(t in desc for t in absent), desc


@pytest.mark.parametrize("debug", ["", "bp_pair=0", "bp_pair=1", "bp_pair=2", "bp_pair=3", "bp_split=0", "bp_split=1", "bp_split=2"])
@pytest.mark.parametrize("seed", range(12))
def test_windows_of_mirror_images_and_shared_views_hold_what_is_read(host, monkeypatch, seed, debug):
    """Random scans, every other one symmetric about the source plane (whose chunks start at the middle layer): no thread of any shape a
    launch may take reads outside its window."""
    from random_geometries import random_config
    cfg = random_config(seed)
    if seed % 2 == 0:
        cfg = cfg.replace(shift_v=0.0, center_z=0.0)
    if cfg.geom == CONE and seed % 3 == 0:
        cfg = cfg.replace(geom=CONE_CURVED)
    if debug:
        monkeypatch.setenv("LEAP_DEBUG", debug)
    rep, desc = window_report(host, cfg)
    assert rep[7] == 0, (rep, desc)


@pytest.mark.parametrize("tiles_x", [1, 3, 7, 8, 9, 16, 21, 64])
def test_the_back_projection_s_order_of_tiles_names_every_tile_once(host, tiles_x):
    for tiles_y in range(1, 34):
        for y in (0, 1, 7, 8):
            assert host.host_check_tile_order(tiles_x, tiles_y, y) == 0, (tiles_y, y)


def test_turns_at_a_handle_s_shared_memory_wait_for_one_another(host):
    """Whatever the streams' handles: 2 is hipStreamPerThread, another stream in every thread, and a destroyed stream's handle may come back as
    another stream's.  A call that returns early leaves its event too; captured turns are ordered within their capture, eager ones apart from them."""
    def turns(streams, captures=None, abandoned=-1):
        n = len(streams)
        out = (C.c_int64 * 3 * n)()
        host.host_shared_turns((C.c_int64 * n)(*streams), (C.c_int64 * n)(*(captures or [0] * n)), n, abandoned, out)
        return [tuple(o) for o in out]

    assert turns([2, 2, 7, 7, 0]) == [(0, 1, 0)] + [(1, 1, 0)] * 4
    assert turns([2, 7, 7], abandoned=0) == [(0, 1, 0), (1, 1, 0), (1, 1, 0)]
    assert turns([7, 5, 6, 5, 7, 7], [0, 11, 11, 12, 0, 0]) == [(0, 1, 0), (0, 2, 1), (2, 2, 1), (0, 2, 1), (1, 1, 0), (1, 1, 0)]
    assert turns([0, 0], [0, -1]) == [(0, 1, 0), (1, 1, 1)]


@pytest.mark.parametrize("nviews,shared", [(2, True), (200, False)])
def test_batches_whose_layers_are_shared_keep_one_volume_s_slabs(host, nviews, shared):
    """Narrow slabs leave waves that share a slab's layers without any; waves of a bundle each take them for the sake of more items per launch."""
    cfg = CTConfig("oblong", CONE, nviews=nviews, arc_deg=360.0, nrows=39, ncols=127, pixel_v=0.9, pixel_u=1.2, nx=100, ny=76, nz=34, voxel_xy=1.0,
                   voxel_z=1.0, sod=450.0, sdd=675.0, shift_v=-0.4)
    h = handle(host, cfg)
    assert ("parts=4" in B.leap_geometry_describe(h, host)) == shared
    plan = (C.c_int64 * 2)()
    host.host_plan_scratch.argtypes = [C.c_void_p, C.c_int, C.c_void_p]
    plans = {}
    for batch in (1, 8, 16, 17):
        host.host_plan_scratch(h, batch, plan)
        plans[batch] = tuple(plan)
    B.leap_geometry_destroy(h, host)
    assert plans[1] == (100, 1) and plans[8] == (100, 8), plans
    assert plans[16] == plans[17] == (100, 8) if shared else plans[16][0] < 100 and plans[16][1] == 16, plans


def test_waves_without_a_block_are_left_out(host):
    """... and with them gone every block still has one wave, the next block the same or the next one."""
    assert host.host_check_waves_for() == 0


def test_calls_on_several_streams_take_slots_of_their_own(host):
    """A stream keeps its slot while there are slots for all; hipStreamPerThread (2) may be another stream each time; a call that takes them all
    waits for each, and each next one for it."""
    def take(streams, slots):
        n = len(streams)
        out = (C.c_int64 * 2 * n)()
        host.host_room_slots((C.c_int64 * n)(*streams), n, slots, out)
        return [tuple(o) for o in out]

    assert take([7, 0, 7, 5, 6, 7, 0], 4) == [(0, 0), (1, 0), (0, 1), (2, 0), (3, 0), (0, 1), (1, 1)]
    assert take([2, 2, 2, 2, 2], 4) == [(0, 0), (1, 0), (2, 0), (3, 0), (0, 1)]
    assert take([3, 4, 5, 3, 4], 2) == [(0, 0), (1, 0), (0, 1), (1, 1), (0, 1)]
    assert take([7, 5, -1, 6, 7], 4) == [(0, 0), (1, 0), (-1, 2), (2, 1), (0, 1)]
    assert take([7, 5, -1, -1, 5, 6, -1], 4) == [(0, 0), (1, 0), (-1, 2), (-1, 1), (1, 1), (2, 1), (-1, 3)]
    assert take([7, 5, -1], 1) == [(0, 0), (0, 1), (-1, 1)]


@pytest.mark.parametrize("geom,n,nz,nrows,nviews,columns", [
    (CONE, 96, 400, 16, 1, True), (CONE, 96, 400, 15, 60, False), (PARALLEL, 96, 400, 22, 1, True), (PARALLEL, 96, 400, 21, 60, False),
    (CONE, 512, 512, 24, 15, False), (CONE, 512, 512, 24, 360, True), (CONE, 512, 512, 32, 1, True), (PARALLEL, 512, 512, 31, 100, False),
    ("upright", 96, 400, 31, 60, False), ("upright", 96, 20, 31, 12, False), ("upright", 96, 20, 31, 15, True), ("upright", 96, 20, 21, 60, False)])
def test_siddon_short_detectors_copy_a_volume_only_where_it_pays(host, geom, n, nz, nrows, nviews, columns):
    """The column-wise forward projection copies the volume, the thread-per-ray kernel reads the few layers its rays cross."""
    par = dict(sod=0.0, sdd=0.0) if geom == PARALLEL else dict(sod=2.0 * n, sdd=3.0 * n)
    cfg = CTConfig("short", CONE if geom == "upright" else geom, nviews=nviews, arc_deg=360.0, nrows=nrows, ncols=n, pixel_v=1.0, pixel_u=1.5,
                   nx=n, ny=n, nz=nz, voxel_xy=1.0, voxel_z=1.0, shift_v=0.2, **par)
    h = handle(host, perturbed_poses(cfg, 5, shift_mm=3.0, upright=True) if geom == "upright" else cfg, B.LEAP_MODEL_SIDDON)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert ("A=columns" in desc) == columns, desc


FEW_TILES = CTConfig("few_tiles", CONE, nviews=203, arc_deg=360.0, nrows=40, ncols=60, pixel_v=1.5, pixel_u=1.6, nx=37, ny=35, nz=27, voxel_xy=1.0,
                     voxel_z=1.0, start_deg=3.0, shift_u=0.3, shift_v=0.3, sod=150.0, sdd=225.0)


@pytest.mark.parametrize("model", [B.LEAP_MODEL_SF, B.LEAP_MODEL_SIDDON])
def test_room_for_the_parts_of_a_back_projection_is_reported(host, monkeypatch, model):
    """scratch= is all the device memory the handle owns beyond its tables; what was not to be had is in the notes, every one of them."""
    def describe(lib):
        h = handle(lib, FEW_TILES, model)
        desc = B.leap_geometry_describe(h, lib)
        B.leap_geometry_destroy(h, lib)
        return desc

    desc = describe(host)
    parts = int(desc.split("+parts(")[1].split(",")[0])
    monkeypatch.setenv("LEAP_DEBUG", "bp_parts=1")
    whole = describe(host)
    one = 4 * parts * FEW_TILES.nx * FEW_TILES.ny * FEW_TILES.nz
    assert "+parts(" not in whole and scratch_bytes(desc) - scratch_bytes(whole) == one * min(16, (64 << 20) // one), (desc, whole)
    if model == B.LEAP_MODEL_SF:                              # (the other's ray table is as large as its scratch)
        monkeypatch.delenv("LEAP_DEBUG")
        host.host_limit_device_allocations.argtypes = [C.c_size_t]
        host.host_limit_device_allocations(100 << 10)
        try:
            poor = describe(host)
        finally:
            host.host_limit_device_allocations(0)
        assert scratch_bytes(poor) == 0 and "forward projection runs on the general kernel" in poor and "no room for the back projection's parts" in poor, poor


@pytest.mark.parametrize("limit,items", [(0, 16), (20 << 20, 8), (5 << 20, 2), (3 << 20, 0)])
def test_flat_scratch_shrinks_to_what_can_be_had(host, limit, items):
    """Two copies of 16 slices of 1 MB where there is room for them, of fewer where there is not, none below two slices."""
    cfg = CTConfig("slice", PARALLEL, nviews=90, arc_deg=180.0, nrows=1, ncols=600, pixel_v=1.0, pixel_u=1.0, nx=500, ny=500, nz=1, voxel_xy=1.0, voxel_z=1.0)
    host.host_limit_device_allocations.argtypes = [C.c_size_t]
    host.host_limit_device_allocations(limit)
    try:
        h = handle(host, cfg)
    finally:
        host.host_limit_device_allocations(0)
    desc = B.leap_geometry_describe(h, host)
    B.leap_geometry_destroy(h, host)
    assert scratch_bytes(desc) == 2 * items * 1000000 and ("note=" in desc) == (items == 0), desc


OWN_LIBRARY = """
import ctypes as C, sys
import numpy as np
sys.path[:0] = [{root!r}, {here!r}]
import test_host_logic as T
from paper_2307_05801_amd import binding as B
lib = C.CDLL(T.LIB)
cfg = T.reduced(T.config(3), 32, nviews=5).replace(nx=19, ny=17, nz=11, nrows=5, ncols=23)
h = T.handle(lib, cfg)
x, y = T.uniform_volume(cfg, 1)[0], np.zeros(cfg.sino_shape, np.float32)
B.leap_project(h, x.ctypes.data, y.ctypes.data, 1, 0, lib)
x2 = np.zeros_like(x)
B.leap_backproject(h, y.ctypes.data, x2.ctypes.data, 1, 0, lib)
assert y.any() and x2.any()
print("done")
"""


def test_calls_through_a_library_that_was_loaded_without_prototypes(host):
    """An address that is passed as a plain integer would be cut to 32 bits."""
    import sys
    res = subprocess.run([sys.executable, "-c", OWN_LIBRARY.format(root=ROOT, here=HERE)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "done" in res.stdout, (res.returncode, res.stderr[-1500:])


def test_no_room_for_parts_is_kept_where_the_general_kernel_runs(host):
    """The cylinder's tables find no room on the device: the back projection has no parts and keeps no memory for them."""
    cfg, seen = FEW_TILES.replace(geom=CONE_CURVED), set()
    for n in range(12):
        host.host_fail_device_allocation(C.c_long(n))
        try:
            h = handle(host, cfg)
        except B.LeapError:
            continue
        finally:
            host.host_fail_device_allocation(C.c_long(-1))
        desc = B.leap_geometry_describe(h, host)
        B.leap_geometry_destroy(h, host)
        general = "AT=general" in desc
        seen.add(general)
        assert not general or scratch_bytes(desc) < 4 << 20, desc            # (the forward scratch alone)
    assert seen == {True, False}


def back_parts(host, h, items):
    """(parts, shape, items at a time, shape one volume takes without parts) of a back projection of `items` volumes."""
    out = (C.c_int32 * 4)()
    host.host_back_parts.argtypes = [C.c_void_p, C.c_int, C.POINTER(C.c_int32)]
    host.host_back_parts(h, items, out)
    return tuple(out)


def test_batches_of_the_gpu_tests_take_parts_in_the_rounds_they_are_meant_to(host):
    from tests.test_gpu_back_parts import CASES as SF_PARTS, ROUNDS, SIDDON as SIDDON_PARTS
    runs = [(n, c, "sf", 3, 3) for n, c in SF_PARTS.items()] + [(n, c, "siddon", 3, 3) for n, c in SIDDON_PARTS.items()]
    runs += [(n, c, m, batch, {7: 4, 21: 16}[batch]) for n, (c, m, batch) in ROUNDS.items()]
    for name, cfg, model, batch, at_once in runs:
        h = handle(host, cfg, B.MODELS[model])
        one, many = back_parts(host, h, 1), back_parts(host, h, batch)
        B.leap_geometry_destroy(h, host)
        assert one[0] > 1 and many == one[:2] + (at_once,) + one[3:], (name, model, one, many)


def parts_scan(kind, nx, ny, nz, nviews, nrows, ncols, pixel_v, pixel_u):
    flat = kind == "parallel"
    far = 0.0 if flat else max(nx, ny) * 1.0
    cfg = CTConfig("parts", {"parallel": PARALLEL, "curved": CONE_CURVED}.get(kind, CONE), nviews=nviews, arc_deg=360.0, nrows=nrows, ncols=ncols,
                   pixel_v=pixel_v / (1.5 if flat else 1.0), pixel_u=pixel_u / (1.5 if flat else 1.0), nx=nx, ny=ny, nz=nz, voxel_xy=1.0, voxel_z=1.0,
                   start_deg=3.0, shift_u=0.3, shift_v=0.0 if kind == "mirror" else 0.3, sod=3.0 * far + 60.0 * (not flat), sdd=4.5 * far + 90.0 * (not flat))
    if kind == "upright":
        return perturbed_poses(cfg, 5, shift_mm=3.0, upright=True)
    return perturbed_poses(cfg, 5, shift_mm=3.0, tilt_rad=0.05) if kind == "tilted" else cfg


@pytest.mark.parametrize("case,shape,alone", [
    (("cone", 106, 60, 26, 332, 26, 105, 1.65, 1.6), 0, 2), (("cone", 23, 69, 64, 53, 65, 67, 1.4, 1.74), 1, 2), (("curved", 31, 99, 18, 92, 24, 86, 1.47, 1.39), 1, 2),
    (("parallel", 35, 33, 84, 149, 130, 36, 1.64, 1.7), 0, 2), (("mirror", 52, 67, 45, 55, 66, 77, 1.15, 1.6), 1, 2), (("upright", 78, 74, 40, 68, 49, 87, 1.34, 1.61), 1, 2)])
def test_windows_of_views_shared_among_workgroups_hold_what_is_read(host, case, shape, alone):
    """Scans whose parts take another shape than one volume's views would within a workgroup."""
    cfg = parts_scan(*case)
    h = handle(host, cfg)
    plan = back_parts(host, h, 1)
    B.leap_geometry_destroy(h, host)
    rep, desc = window_report(host, cfg)
    assert plan[0] > 1 and plan[1] == shape and plan[3] == alone and rep[7] == 0, (plan, rep, desc)


@pytest.mark.parametrize("case,shape,alone", [
    (("cone", 66, 77, 46, 54, 47, 94, 1.67, 1.52), 0, 1), (("curved", 28, 62, 29, 108, 42, 91, 1.49, 1.61), 0, 1), (("parallel", 72, 24, 14, 162, 15, 80, 0.73, 1.17), 0, 1),
    (("upright", 44, 47, 11, 207, 11, 69, 1.35, 1.58), 0, 1), (("tilted", 21, 38, 58, 67, 54, 49, 1.04, 1.41), 0, 0), (("tilted", 37, 35, 27, 203, 76, 100, 0.74, 0.9), 2, 2)])
def test_siddon_views_shared_among_workgroups_match_oracle_on_cpu(host, oracle_mod, case, shape, alone):
    """The shape that the parts take, re-enacted: every window and slot holds what is read and written, and the result is the oracle's."""
    cfg = parts_scan(*case)
    y = uniform_sinogram(cfg, 6)[0]
    h = handle(host, cfg, B.LEAP_MODEL_SIDDON)
    desc, plan = B.leap_geometry_describe(h, host), back_parts(host, h, 1)
    out, rep = np.full(cfg.vol_shape, np.nan, np.float32), (C.c_int64 * 4)()
    run = host.host_md_backproject_tiled if case[0] == "tilted" else host.host_sd_backproject_tiled
    bad = run(h, y.ctypes.data, out.ctypes.data, rep)
    B.leap_geometry_destroy(h, host)
    assert plan[0] > 1 and plan[1] == shape and plan[3] == alone and bad == 0, (plan, bad, list(rep), desc)
    ref = oracle_mod.siddon.backproject(cfg, y)
    assert rel_l2(out, ref) <= TOL and np.abs(out - ref).max() <= 2e-5 * np.abs(ref).max(), desc       # (the tilted re-enactments' tolerance)
