"""The forward on small detectors (8x8 rays a block, each chunk of samples shared
by its four wavefronts): ragged detectors, single pixels, chunk boxes that touch
the grid's faces or do not fit LDS, the last size that is split against the
first that is not, and one view's values whatever is launched with it.  The bar
is the existing 1e-5 of max|ref|."""
import math

import numpy as np
import pytest
import torch

import synth
from synth import Geom

pytestmark = pytest.mark.gpu


def project(dp, g, vol, angles, poses):
    t = [torch.tensor(np.ascontiguousarray(a), dtype=d, device="cuda:0")
         for a, d in ((angles, torch.float64), (poses, torch.float64), (vol, torch.float32))]
    return dp.project_fwd(g, *t).cpu().numpy()


# volume, voxel mm, detector, pixel mm, views
@pytest.mark.parametrize("n,h,nu,nv,du,V", [
    ((1, 1, 1), 4.0, 9, 7, 1.0, 2), ((5, 4, 3), 6.0, 1, 1, 1.0, 1), ((40, 36, 33), 1.5, 8, 9, 6.0, 1),
    ((40, 36, 33), 1.5, 63, 65, 1.6, 3), ((41, 35, 33), 1.5, 17, 15, 4.0, 2), ((64, 64, 64), 1.0, 12, 12, 25.0, 2),
    ((33, 64, 40), 0.3, 40, 20, 1.2, 2), ((24, 24, 24), 3.0, 48, 16, 3.0, 256), ((24, 24, 24), 3.0, 12, 9, 9.0, 769)])
def test_small_launches(dp, oracle, n, h, nu, nv, du, V):
    g = Geom(*n, h, 1.1 * h, 0.9 * h, nu, nv, du, du, off_u=0.5, off_v=-0.25)
    rng = synth.rng_for(1000 + nu + V)
    vol = rng.uniform(0, 0.05, g.vol_shape).astype(np.float32)
    angles = rng.uniform(0, 2 * math.pi, V)
    poses = synth.random_poses(V, 2.0, 60.0, rng)
    ref = oracle.project_fwd(g, angles, poses, vol)
    assert np.abs(ref).max() > 0
    assert np.abs(project(dp, g, vol, angles, poses) - ref).max() <= 1e-5 * np.abs(ref).max()


def test_source_inside_and_a_voxel_without_a_number(dp, oracle):
    g = Geom(24, 24, 24, 2.0, 2.0, 2.0, 20, 18, 4.0, 4.0, sad=20.0, sdd=40.0)
    rng = synth.rng_for(1100)
    vol = rng.uniform(0, 0.05, g.vol_shape).astype(np.float32)
    angles, poses = rng.uniform(0, 2 * math.pi, 2), synth.random_poses(2, 2.0, 20.0, rng)
    ref = oracle.project_fwd(g, angles, poses, vol)
    got = project(dp, g, vol, angles, poses)
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
    vol[0, 12, 12] = np.nan
    hit = np.isnan(project(dp, g, vol, angles, poses))
    assert np.array_equal(hit, np.isnan(oracle.project_fwd(g, angles, poses, vol)))



# 144 tiles of 16x16 are split, 145 not (boxes with and without room for the wide slice pitch)
@pytest.mark.parametrize("n,h,nu,nv,du,V", [((48, 48, 48), 2.0, 192, 192, 0.9, 2), ((37, 50, 41), 2.5, 193, 191, 0.9, 2),
                                            ((64, 64, 20), 1.0, 2320, 9, 0.1, 2), ((48, 48, 48), 2.0, 144, 260, 1.1, 3)])
def test_largest_split_and_smallest_whole(dp, oracle, n, h, nu, nv, du, V):
    test_small_launches(dp, oracle, n, h, nu, nv, du, V)


def test_a_view_does_not_depend_on_its_launch(dp):
    g = Geom(96, 96, 96, 1.0, 1.0, 1.0, 192, 192, 0.9, 0.9)
    rng = synth.rng_for(1200)
    vol = synth.ellipsoid_phantom(96, 1.0, 8, rng)
    angles, poses = rng.uniform(0, 2 * math.pi, 9), synth.random_poses(9, 5.0, 5.0, rng)
    every = project(dp, g, vol, angles, poses)
    for i in (0, 4, 8):
        assert np.array_equal(project(dp, g, vol, angles[i:i + 1], poses[i:i + 1])[0], every[i])


# rays far apart, whose chunks are not worth staging (every fourth sample per
# wavefront straight from the volume), split and whole; rays close together
SPACINGS = [((100, 97, 95), 1.5, 50, 47, 6.6, 3), ((160, 150, 140), 0.9, 100, 97, 3.0, 2),
            ((160, 150, 140), 0.9, 200, 190, 3.0, 2), ((33, 30, 28), 4.5, 160, 157, 1.2, 2)]


@pytest.mark.parametrize("n,h,nu,nv,du,V", SPACINGS)
def test_ray_spacings(dp, oracle, n, h, nu, nv, du, V):
    test_small_launches(dp, oracle, n, h, nu, nv, du, V)


def test_batches_of_ray_spacings(dp):
    rng = synth.rng_for(1300)
    prs, want = [], []
    for n, h, nu, nv, du, V in SPACINGS:
        g = Geom(*n, h, h, h, nu, nv, du, du)
        t = [torch.tensor(np.ascontiguousarray(a), dtype=d, device="cuda:0")
             for a, d in ((rng.uniform(0, 2 * math.pi, V), torch.float64), (synth.random_poses(V, 2.0, 9.0, rng), torch.float64),
                          (rng.uniform(0, 0.05, g.vol_shape), torch.float32))]
        want.append(dp.project_fwd(g, *t))
        prs.append(dict(geom=g, angles=t[0], poses=t[1], vol=t[2], proj=torch.zeros_like(want[-1])))
    dp.project_fwd_batch(prs, variant=1)
    for p, w in zip(prs, want):
        assert torch.equal(p["proj"], w)
