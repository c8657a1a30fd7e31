"""Footprint gathers and scatter at the edges of their pixel windows: windows
of one quad, of several quads, taller than five rows, detectors narrower than a
quad, and pixels of weight zero that hold no number.  Same bars as
test_gpu_footprint.py."""
import math

import numpy as np
import pytest

import synth
from synth import Geom
from test_gpu_parity import check_grads, check_values, f32, f64

pytestmark = pytest.mark.gpu

# voxel widths on the detector: 1.5 px (one quad), 5.5 px (several quads, row
# counts around five), 9 px (pixel by pixel); detectors of 3, 4 and 5 columns;
# columns and rows past the detector's edges in all of them
CASES = {
    "one-quad": Geom(21, 18, 19, 1.0, 1.0, 1.0, 23, 21, 1.0, 1.0, off_u=2.5, off_v=-1.25),
    "quads": Geom(11, 10, 9, 2.0, 2.0, 2.0, 52, 47, 0.55, 0.55, off_u=-3.5),
    "pixels": Geom(9, 8, 7, 2.0, 2.0, 2.0, 70, 61, 0.33, 0.33, off_v=4.0),
    "tall": Geom(10, 9, 8, 1.0, 1.0, 3.0, 16, 60, 1.0, 0.6),
    "nu3": Geom(12, 11, 10, 1.0, 1.0, 1.0, 3, 14, 2.0, 1.0),
    "nu4": Geom(12, 11, 10, 1.0, 1.0, 1.0, 4, 1, 2.0, 9.0),
    "nu5": Geom(70, 5, 17, 0.5, 1.0, 1.0, 5, 2, 4.0, 5.0),
}


@pytest.mark.parametrize("kind", ["sf", "dd"])
@pytest.mark.parametrize("name", list(CASES))
def test_windows_match_oracle(dp, oracle, name, kind):
    g, V = CASES[name], 3
    rng = synth.rng_for(760 + list(CASES).index(name))
    vol = rng.uniform(0.0, 0.05, g.vol_shape).astype(np.float32)
    vol[:, : g.ny // 2, : g.nx // 3] = 0.0  # voxels without a footprint to scatter
    angles, poses = rng.uniform(0, 2 * math.pi, V), synth.random_poses(V, 2.0, 9.0, rng)
    a, p = f64(angles), f64(poses)
    img = rng.standard_normal((V, g.nv, g.nu)).astype(np.float32)
    e = rng.standard_normal(g.vol_shape).astype(np.float32)
    check_values(f"{name} {kind} project", dp.fp_project(g, a, p, f32(vol), kind).cpu().numpy(),
                 oracle.fp_project(g, angles, poses, vol, kind))
    check_values(f"{name} {kind} backproject", dp.fp_backproject(g, a, p, f32(img), kind).cpu().numpy(),
                 oracle.fp_backproject(g, angles, poses, img, kind))
    check_grads(f"{name} {kind} project_grad_pose",
                dp.fp_project_grad_pose(g, a, p, f32(vol), f32(img), kind).cpu().numpy(),
                oracle.fp_project_grad_pose(g, angles, poses, vol, img, kind))
    check_grads(f"{name} {kind} backproject_grad_pose",
                dp.fp_backproject_grad_pose(g, a, p, f32(img), f32(e), kind).cpu().numpy(),
                oracle.fp_backproject_grad_pose(g, angles, poses, img, e, kind))


@pytest.mark.parametrize("value", [math.inf, math.nan])
@pytest.mark.parametrize("kind", ["sf", "dd"])
def test_pixel_without_a_number_reaches_its_voxels_only(dp, oracle, kind, value):
    g = CASES["one-quad"]
    rng = synth.rng_for(780)
    angles, poses = np.array([0.4]), synth.random_poses(1, 1.0, 4.0, rng)
    img = rng.standard_normal((1, g.nv, g.nu)).astype(np.float32)
    img[0, 9, 11] = 0.0
    clean = dp.fp_backproject(g, f64(angles), f64(poses), f32(img), kind).cpu().numpy()
    img[0, 9, 11] = value
    got = dp.fp_backproject(g, f64(angles), f64(poses), f32(img), kind).cpu().numpy()
    ind = np.zeros_like(img)
    ind[0, 9, 11] = 1.0
    w = oracle.fp_backproject(g, angles, poses, ind, kind)
    away, hit = w == 0.0, w > 1e-4 * w.max()
    # a voxel whose footprint ends within rounding of the pixel's edge may touch it
    assert np.mean(np.isfinite(got[away])) > 0.999 and not np.isfinite(got[hit]).any()
    ok = away & np.isfinite(got)
    np.testing.assert_array_equal(got[ok], clean[ok])


@pytest.mark.parametrize("value", [math.inf, -math.inf, math.nan])
@pytest.mark.parametrize("kind", ["sf", "dd"])
@pytest.mark.parametrize("name", ["one-quad", "quads"])
def test_voxel_without_a_number_reaches_its_pixels_only(dp, oracle, name, kind, value):
    g = CASES[name]
    rng = synth.rng_for(790)
    angles, poses = np.array([0.4, 2.0]), synth.random_poses(2, 1.0, 4.0, rng)
    vol = rng.uniform(0.0, 0.05, g.vol_shape).astype(np.float32)
    at = (g.nz // 2, g.ny // 2 - 1, g.nx // 2 + 1)
    vol[at] = 0.0
    clean = dp.fp_project(g, f64(angles), f64(poses), f32(vol), kind).cpu().numpy()
    vol[at] = value
    got = dp.fp_project(g, f64(angles), f64(poses), f32(vol), kind).cpu().numpy()
    ind = np.zeros_like(vol)
    ind[at] = 1.0
    w = oracle.fp_project(g, angles, poses, ind, kind)
    away, hit = w == 0.0, w > 1e-4 * w.max()
    assert hit.sum() >= 2
    # a footprint that ends within rounding of a pixel's edge may touch that pixel
    rim = away & ~np.isfinite(got)
    assert rim.sum() <= 2
    assert (np.isnan(got[hit]) if math.isnan(value) else got[hit] == value).all()
    ok = away & ~rim
    # (FP32 atomics: the last bits depend on the order of the sums)
    assert np.abs(got[ok] - clean[ok]).max() <= 1e-5 * np.abs(clean).max()


# blocks that take several views each: 100 blocks (20 share the views of a brick, so
# that 47 views make two or three a block) and 2048 (every block takes them all)
@pytest.mark.parametrize("n,V", [((70, 40, 40), 47), ((64, 256, 256), 3)])
@pytest.mark.parametrize("kind", ["sf", "dd"])
def test_gradient_of_a_view_does_not_depend_on_its_launch(dp, oracle, kind, n, V):
    g = Geom(*n, 1.0, 1.0, 1.0, 61, 49, 2.0, 2.0, off_u=1.5)
    rng = synth.rng_for(795)
    angles, poses = rng.uniform(0, 2 * math.pi, V), synth.random_poses(V, 2.0, 9.0, rng)
    vol, e = f32(rng.uniform(0.0, 0.05, g.vol_shape).astype(np.float32)), f32(rng.standard_normal(g.vol_shape).astype(np.float32))
    img = f32(rng.standard_normal((V, g.nv, g.nu)).astype(np.float32))
    a, p = f64(angles), f64(poses)
    fwd = dp.fp_project_grad_pose(g, a, p, vol, img, kind).cpu().numpy()
    back = dp.fp_backproject_grad_pose(g, a, p, img, e, kind).cpu().numpy()
    for v in range(V):
        one = slice(v, v + 1)
        np.testing.assert_array_equal(dp.fp_project_grad_pose(g, a[one], p[one], vol, img[one], kind).cpu().numpy(), fwd[one])
        np.testing.assert_array_equal(dp.fp_backproject_grad_pose(g, a[one], p[one], img[one], e, kind).cpu().numpy(), back[one])
    last = slice(V - 1, V)
    if n[0] == 70:
        check_grads(f"{kind} project_grad_pose", fwd[last],
                    oracle.fp_project_grad_pose(g, angles[last], poses[last], vol.cpu().numpy(), img[last].cpu().numpy(), kind))
        check_grads(f"{kind} backproject_grad_pose", back[last],
                    oracle.fp_backproject_grad_pose(g, angles[last], poses[last], img[last].cpu().numpy(), e.cpu().numpy(), kind))
