"""Kernels at the sizes where their work split can go wrong: partial matrix
tiles and workgroups, scans over one round and more, cells at block borders
(needs an MI355X)."""

import math

import numpy as np
import pytest
import torch

import oracle
from synthetic.scenes import Intrinsics, look_at

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mlp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_7194_amd.mlp as M

    M.T.lib()
    return M


@pytest.mark.parametrize("batch", [1, 31, 32, 33, 127, 129, 2049])
def test_training_batches_around_a_tile(mlp, batch):
    """Loss and gradient of batches that leave the last 32-sample tile or
    128-sample workgroup partly empty, drawn from the middle of a visiting
    order that wraps around.  Gate: the repository's (the bfloat16 errors can
    flip where float and double straddle a rounding boundary)."""
    rng = np.random.default_rng(batch)
    n, first, perm = 3001, 2900, (1234, 567)
    assert math.gcd(perm[0], n) == 1
    x = np.column_stack([rng.uniform(0.3, 3, n), rng.uniform(0, 1, n), rng.uniform(0, 1, n),
                         rng.uniform(0, 0.7, n)]).astype(np.float32).astype(np.float64)
    r = (0.0015 * x[:, 0] ** 2 * rng.normal(0, 1, n)).astype(np.float32)
    p = mlp.init_params(7)
    p[mlp.OFF_W3:mlp.OFF_B3] += rng.normal(0, 0.3, 32)
    p = oracle.bf16(p)
    loss, grad = mlp.loss_grad(mlp.params_from_values(p), torch.tensor(x, dtype=torch.float32, device="cuda"),
                               torch.tensor(r, device="cuda"), first, batch, perm)
    torch.cuda.synchronize()
    at = (perm[0] * ((first + np.arange(batch)) % n) + perm[1]) % n
    oloss, og = oracle.mlp_loss_grad(p, x[at], r[at].astype(np.float64), round_bf16=True)
    g = grad.cpu().numpy().astype(np.float64)
    assert abs(loss.item() - oloss) <= 1e-4 * abs(oloss) + 1e-6
    assert np.abs(g - og).max() <= 1e-3 * np.abs(og).max()


@pytest.mark.parametrize("W,H", [(7, 5), (640, 420)])
def test_samples_are_collected_in_pixel_order(mlp, W, H):
    """Rows appended to a running total, in pixel order, over one scan round of
    1024 workgroups and over more; rows beyond the capacity are counted only."""
    rng = np.random.default_rng(W)
    K = Intrinsics(0.9 * W + 20.0, 0.9 * W + 20.0, W / 2.0, H / 2.0, W, H)
    d = (1.0 + 0.1 * rng.random((H, W))).astype(np.float32)
    d[rng.random((H, W)) < 0.1] = 0.0
    pose = np.hstack([np.eye(3), np.zeros((3, 1))])
    vert = rng.random((H, W, 4)).astype(np.float32) + np.float32(0.5)
    vert[rng.random((H, W)) < 0.2] = 0.0
    depth, vertex = torch.from_numpy(d).cuda(), torch.from_numpy(vert).cuda()
    feat, valid = mlp.features(depth, K)
    ok = (valid.cpu().numpy().reshape(H, W) > 0) & (vert[..., 3] > 0) & (d > 0)
    n = int(ok.sum())
    col = mlp.SampleCollector(max(2 * n - 3, 1), W, H)
    col.add(depth, K, pose, vertex)
    col.add(depth, K, pose, vertex)
    torch.cuda.synchronize()
    assert int(col.count.item()) == 2 * n
    x, r = (t.cpu().numpy() for t in col.samples())
    ef = feat.cpu().numpy().reshape(H, W, 4)[ok]
    er = (d.astype(np.float64) - vert[..., 2].astype(np.float64))[ok].astype(np.float32)
    m = len(r)
    assert m == max(2 * n - 3, 1) or n < 2
    assert np.array_equal(x, np.concatenate([ef, ef])[:m]) and np.array_equal(r, np.concatenate([er, er])[:m])
