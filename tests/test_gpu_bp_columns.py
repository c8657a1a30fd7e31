"""Voxel-driven back-projection at its column lengths (8 voxels, and 32 from 2048
blocks of 64 x 4 columns on) and through each of its column forms: inside the
detector, off it, across its edge, tilted beyond the depth series, around the
source.  The bar is the existing 1e-5 of max|ref|."""
import numpy as np
import pytest
import torch

import synth
from synth import Geom

pytestmark = pytest.mark.gpu

# (volume, detector, rotation range in degrees): columns all inside; most off a
# small detector; tilts that exceed the depth series; the source in the volume
FORMS = {
    "inside": (dict(hx=0.5, hz=0.5, nu=90, du=2.5), 3.0),
    "truncated": (dict(hx=2.0, hz=2.0, nu=21, du=2.0), 5.0),
    "tilted": (dict(hx=1.5, hz=1.5, nu=60, du=2.5), 80.0),
    "around": (dict(hx=2.0, hz=2.0, nu=40, du=2.0, sad=20.0, sdd=40.0), 20.0),
}


def inputs(form, nx, ny, nz, V):
    o, deg = FORMS[form]
    src = dict(sad=o["sad"], sdd=o["sdd"]) if "sad" in o else {}
    g = Geom(nx, ny, nz, o["hx"], o["hx"], o["hz"], o["nu"], o["nu"] - 3, o["du"], o["du"], off_u=0.75, **src)
    rng = synth.rng_for(900 + nx + nz)
    angles = rng.uniform(0, 2 * np.pi, V)
    poses = synth.random_poses(V, 4.0, deg, rng)
    proj = rng.standard_normal((V, g.nv, g.nu)).astype(np.float32)
    return g, angles, poses, proj


def run(dp, g, angles, poses, proj, mode):
    t = [torch.tensor(np.ascontiguousarray(a), dtype=d, device="cuda:0")
         for a, d in ((angles, torch.float64), (poses, torch.float64), (proj, torch.float32))]
    return dp.backproject(g, *t, weight_mode=mode).cpu().numpy()


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("nx,ny,nz", [(63, 3, 7), (65, 5, 9), (64, 4, 33)])
@pytest.mark.parametrize("mode", [0, 1])
def test_short_columns(dp, oracle, form, nx, ny, nz, mode):
    args = inputs(form, nx, ny, nz, 4)
    ref = oracle.backproject(*args, weight_mode=mode)
    assert np.abs(run(dp, *args, mode) - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("form,h", [("inside", 0.06), ("truncated", 0.5), ("tilted", 0.2), ("around", 0.2)])
def test_long_columns(dp, oracle, form, h):
    nx, ny, nz = 65, 130, 995
    g, angles, poses, proj = inputs(form, nx, ny, nz, 3)
    o = FORMS[form][0]
    g = Geom(nx, ny, nz, 10 * h, 5 * h, h, g.nu, g.nv, o["du"], o["du"], off_u=0.75,
             **(dict(sad=o["sad"], sdd=o["sdd"]) if "sad" in o else {}))
    ids = np.random.default_rng(3).integers(0, nx * ny * nz, 40000)
    ids = np.concatenate([ids, [0, nx * ny * nz - 1], np.arange(nz) * nx * ny + nx * ny - 1]).astype(np.int64)
    ref = oracle.backproject_voxels(g, angles, poses, proj, ids, 1)
    got = run(dp, g, angles, poses, proj, 1).reshape(-1)[ids]
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


def test_pixel_without_a_number_reaches_its_own_voxels(dp):
    g, angles, poses, proj = inputs("truncated", 65, 12, 40, 2)
    want = run(dp, g, angles, poses, proj, 0)
    proj[1, 9, 10] = np.nan
    got = run(dp, g, angles, poses, proj, 0)
    hit = np.isnan(got)
    assert 0 < hit.sum() < got.size // 4 and np.array_equal(got[~hit], want[~hit])
