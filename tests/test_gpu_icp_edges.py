"""The ICP solve at its limits: accuracy of the eigen-decomposition over many
systems, and systems with non-finite entries (needs an MI355X)."""

import numpy as np
import pytest
import torch

from oracle import icp as O
from synthetic import Intrinsics

pytestmark = pytest.mark.gpu

IDENTITY = np.hstack([np.eye(3), np.zeros((3, 1))])


@pytest.fixture(scope="module")
def tsdf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_7194_amd as m

    m.lib()
    return m


def test_solution_residual_over_random_systems(tsdf):
    """Without a threshold and without scaling x solves C x = b, and its
    residual relative to |C| |x| is the error that the eigen-decomposition
    leaves.  Four sweeps of five rounds are twenty roundings of 2^-53 per
    direction, sqrt(20) 2^-53 = 5e-16 together; the median over the systems is
    free of those that the sweeps' stopping rule (1e-13) dominates."""
    K = Intrinsics(20.0, 20.0, 7.5, 3.5, 16, 8)
    icp = tsdf.Icp(K, 100.0, 0.0, -1.0, False)
    res = []
    for seed in range(150):
        rng = np.random.default_rng(seed)
        depth = torch.from_numpy(rng.uniform(0.5, 1.5, (8, 16)).astype(np.float32)).cuda()
        MV = np.ones((8, 16, 4), np.float32)
        MV[..., :3] = rng.normal(size=(8, 16, 3))
        MN = np.ones((8, 16, 4), np.float32)
        n = rng.normal(size=(8, 16, 3))
        MN[..., :3] = n / np.linalg.norm(n, axis=-1, keepdims=True)
        icp.run(depth, torch.from_numpy(MV).cuda(), torch.from_numpy(MN).cuda(), IDENTITY, IDENTITY, 1)
        torch.cuda.synchronize()
        g = icp.result(0)
        assert g["N"] >= 20 and g["kept"] == 6
        r = g["C"].astype(np.longdouble) @ g["x"].astype(np.longdouble) - g["b"]
        res.append(float(np.linalg.norm(r.astype(np.float64)) / (np.linalg.norm(g["C"], 2) * np.linalg.norm(g["x"]))))
    print(f"[icp] solution residual: median {np.median(res):.2e}, 90 % {np.quantile(res, 0.9):.2e}, "
          f"largest {max(res):.2e}", flush=True)
    assert np.median(res) <= 5e-16


@pytest.mark.parametrize("shrink", [False, True])
@pytest.mark.parametrize("at", [5, -1])
@pytest.mark.parametrize("normal", [(1.0, 0.0, 0.0), (1.0, 1.0, 0.0), (0.0, 1.0, -1.0)])
def test_infinite_model_normal(tsdf, normal, at, shrink):
    """A model normal with infinite components passes the rejection (inf >= inf).
    Without scaling, every entry of the system that does not hold one of its
    infinite terms stays the finite sum, and all six eigenvalues are written:
    the sweeps cannot start, so they are the system's diagonal, in the order of
    an insertion sort.  With scaling the matrix has no entry left to rely on, but
    the eigenvalues are still its diagonal."""
    K = Intrinsics(20.0, 20.0, 7.5, 3.5, 16, 8)
    rng = np.random.default_rng(3)
    depth = (1.0 + 0.01 * rng.random((8, 16))).astype(np.float32)
    v, n, ok = O.live_points(depth, K.as_tuple())
    MV, MN = np.ones((8, 16, 4), np.float32), np.ones((8, 16, 4), np.float32)
    MV[..., :3] = v + 0.01 * rng.normal(size=v.shape)
    with np.errstate(invalid="ignore"):
        MN[..., :3] = n / np.linalg.norm(n, axis=-1, keepdims=True)
    agrees = ((n * np.array(normal) > 0) | (np.array(normal) == 0)).all(-1)
    one = np.argwhere(ok & agrees)[at]   # a pixel whose normal agrees with it
    MN[one[0], one[1], :3] = [x * np.inf if x else 0.0 for x in normal]
    params = O.IcpParams(dist_max=1.0, cos_min=0.5, theta=-1.0, shrink=shrink)
    with np.errstate(invalid="ignore"):
        p, q, nn, _ = O.associate(depth, K.as_tuple(), MV, MN, IDENTITY, IDENTITY, params)
        g = np.concatenate([O._cross(p, nn), nn], 1)
        C = np.array([[(g[:, a] * g[:, b]).sum() for b in range(6)] for a in range(6)])
        b = -np.array([(g[:, a] * O._dot(p - q, nn)).sum() for a in range(6)])
    assert len(p) > 50 and not np.isfinite(C).all()
    icp = tsdf.Icp(K, 1.0, 0.5, -1.0, shrink)
    icp.results.fill_(-7.0)
    icp.run(torch.from_numpy(depth).cuda(), torch.from_numpy(MV).cuda(), torch.from_numpy(MN).cuda(), IDENTITY,
            IDENTITY, 1)
    torch.cuda.synchronize()
    r = icp.result(0)
    assert r["N"] == len(p)
    if not shrink:
        for got, want in ((r["C"], C), (r["b"], b)):
            fin = np.isfinite(want)
            assert np.array_equal(np.isnan(got), np.isnan(want))
            assert np.abs(got[fin] - want[fin]).max(initial=0.0) <= 1e-9 * np.abs(want[fin]).max(initial=1.0)
            assert np.array_equal(got[~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)])
    want = [float(x) for x in np.diag(r["C"]) / r["N"]]
    for e in range(1, 6):
        f = e
        while f > 0 and want[f - 1] > want[f]:
            want[f - 1], want[f] = want[f], want[f - 1]
            f -= 1
    assert np.array_equal(r["lam"], np.array(want), equal_nan=True)
