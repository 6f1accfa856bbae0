"""The tiled back projections of one volume per workgroup without shared views, which large scans take, on small ragged scans (that leave
the chip idle and would share their views): both models, every kind of detector, against the oracle; the same bits on every call."""
import numpy as np
import pytest

from synthetic import perturbed_poses, uniform_sinogram
from synthetic.configs import CONE, CONE_CURVED
from tests import test_gpu_parity as sf
from tests import test_gpu_siddon as siddon
from tests.random_geometries import random_config, random_tilted_scan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    return torch


def curved(cfg):
    return cfg.replace(geom=CONE_CURVED) if cfg.geom == CONE else cfg


CASES = [("sf", name, make) for name, _, make in sf.SMALL_CASES]
CASES += [("sf", f"upright_{seed}", lambda seed=seed: perturbed_poses(random_config(seed).replace(geom=CONE, shift_v=0.0), seed, shift_mm=2.0, upright=True))
          for seed in (2, 5, 8)]
CASES += [("sf", f"random_{seed}", lambda seed=seed: random_config(seed)) for seed in range(12)]
CASES += [("sf", f"random_curved_{seed}", lambda seed=seed: curved(random_config(seed))) for seed in (1, 2, 5, 7)]
CASES += [("siddon", name, make) for name, _, make in siddon.SMALL_CASES]
CASES += [("siddon", name, make) for name, make in siddon.UPRIGHT_MODULAR_CASES + siddon.TILTED_FAST_CASES]
CASES += [("siddon", f"random_{seed}", lambda seed=seed: siddon.off_face(random_config(seed))) for seed in range(12)]
CASES += [("siddon", f"random_tilted_{seed}", lambda seed=seed: random_tilted_scan(seed)) for seed in range(8)]
# one layer, voxels of too many pixels, windows that fit no shape: the general kernels
GENERAL = {"c1_full", "fan", "fine_detector", "curved_close_source", "steep_thin_slices", "random_7", "random_8", "random_11", "random_curved_7",
           "upright_8"}


@pytest.mark.parametrize("model,name,make", CASES, ids=[f"{c[0]}-{c[1]}" for c in CASES])
def test_one_volume_per_workgroup(torch_mod, oracle_mod, monkeypatch, model, name, make):
    from paper_2307_05801_amd import Geometry
    cfg = make()
    monkeypatch.setenv("LEAP_DEBUG", "bp_split=-1,bp_pair=-1")
    geo = Geometry(cfg, model=model)
    desc = geo.describe()
    print(f"[gpu] {model} {name}: {desc}", flush=True)
    assert not any(s in desc for s in ("+split", "+pairs", "+mirror")), desc
    assert ("AT=tiled" in desc) != (name in GENERAL), desc
    y = uniform_sinogram(cfg, 77, batch=2)
    yt = torch_mod.from_numpy(y).cuda()
    out = geo.backproject(yt)
    oracle = oracle_mod if model == "sf" else oracle_mod.siddon
    for b in range(2):
        want = oracle.backproject(cfg, y[b])
        assert sf.rel_l2(out[b].cpu().numpy(), want) <= sf.TOL                   # the parity tests' tolerances
        assert np.abs(out[b].cpu().numpy() - want).max() <= 2e-5 * np.abs(want).max()
    assert torch_mod.equal(out, geo.backproject(yt))
    geo.close()

