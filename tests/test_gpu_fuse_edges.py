"""Fusion's pixel decisions where single precision can decide little: voxels a
few voxel sizes from the camera, extreme focal lengths (needs an MI355X)."""

import numpy as np
import pytest
import torch

import oracle
from synthetic.scenes import Intrinsics, look_at
from tests.parity import Kvec, compare_volumes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tsdf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_7194_amd as m

    m.lib()
    return m


def fuse_both(tsdf, K, depth, pose, dims, vs, origin, coeff):
    gv = tsdf.Volume(dims, vs, origin, 4.0, 1 << 14, 1 << 15, 0, 1e-4, K.width, K.height)
    ov = oracle.OracleVolume(dims, vs, origin, 4.0, capacity_blocks=1 << 14)
    st = ov.integrate(depth, Kvec(K), pose, coeff=coeff)
    gv.integrate(torch.from_numpy(depth).cuda(), K, pose, coeff=coeff)
    gst = gv.stats()
    assert gst["frame_updates"] == st["updates"] and gst["frame_new_blocks"] == st["new_blocks"]
    assert gst["status_flags"] == 0
    compare_volumes(gv, ov)
    return st["updates"]


@pytest.mark.parametrize("near,far", [(0.3, 3.0), (2.0, 12.0), (6.0, 30.0), (40.0, 90.0)])
@pytest.mark.parametrize("fx", [9.0, 60.0, 900.0])
def test_voxels_close_to_the_camera(tsdf, near, far, fx):
    """Depths of `near` to `far` voxels, each pixel its own, seen from inside the
    volume: the voxels the frame updates are those of the double-precision
    decisions, in front of the camera and about its plane."""
    W, H, vs = 97, 61, 0.01
    K = Intrinsics(fx, 1.1 * fx, 47.3, 30.6, W, H)
    rng = np.random.default_rng(int(10 * near + fx))
    depth = (vs * rng.uniform(near, far, (H, W))).astype(np.float32)
    pose = look_at((0.013, -0.027, 0.009), (0.4, 0.3, 0.5))
    # (900 pixels focal length: a beam a few voxels wide, at 0.3 to 3 voxels none)
    assert fuse_both(tsdf, K, depth, pose, (192, 192, 192), vs, (-0.96, -0.96, -0.96), 0.05) > (50 if fx < 900 else -1)


@pytest.mark.parametrize("fx,z", [(3e4, 0.3), (1e20, 0.3), (1e33, 0.3), (1e33, 0.0123), (1e300, 0.3)])
def test_focal_lengths_past_single_precision(tsdf, fx, z):
    """Only the voxels on the camera's axis fall into the image (their centres lie
    on it exactly: dyadic sizes), whatever the focal length."""
    W, H, vs = 16, 12, 1.0 / 64
    K = Intrinsics(fx, fx, 7.5, 5.5, W, H)
    pose = np.hstack([np.eye(3), np.array([[0.5 * vs], [0.5 * vs], [0.5 * vs]])])
    depth = np.full((H, W), z, np.float32)
    assert 3 <= fuse_both(tsdf, K, depth, pose, (64, 64, 64), vs, (-0.5, -0.5, 0.0), 0.01) <= 9
