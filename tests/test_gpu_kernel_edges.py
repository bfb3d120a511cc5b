"""Kernels at the sizes where their work split can go wrong: partial matrix
tiles and workgroups, scans over one round and more, cells at block borders
(needs an MI355X)."""

import math

import numpy as np
import pytest
import torch

import oracle
from synthetic.configs import sequence_frame, small_orbit
from synthetic.scenes import Intrinsics, look_at
from tests.test_gpu_mesh import compare_meshes, gpu_mesh, load_both
from tests.parity import CHI, Kvec, compare_raycast, compare_volumes, gpu_volume_for, oracle_volume_for

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


@pytest.fixture(scope="module")
def tsdf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_7194_amd as m

    m.lib()
    return m


@pytest.mark.parametrize("W,H", [(60, 45), (24, 18), (13, 9)])
def test_tiles_with_more_blocks_than_their_list(tsdf, W, H):
    """Frames whose pixels are up to four blocks wide: a 16x16-pixel tile
    reaches from some hundred blocks to several times the 1024 its list holds
    (and its last round holds any number)."""
    spec = small_orbit(width=W, height=H, n_frames=2, G=512, vs=0.004)
    gv, ov = gpu_volume_for(spec), oracle_volume_for(spec)
    for k in range(2):
        d, p = sequence_frame(spec, k)
        st = ov.integrate(d.numpy(), Kvec(spec.K), p)
        gv.integrate(d.cuda(), spec.K, p)
        gst = gv.stats()
        assert gst["frame_updates"] == st["updates"] and gst["frame_new_blocks"] == st["new_blocks"]
        assert gst["status_flags"] == 0
    stats = compare_volumes(gv, ov)
    assert stats["blocks"] > 800


@pytest.mark.parametrize("z", [0.125, 1.0])
@pytest.mark.parametrize("shift", [0.0, 0.5])
def test_voxel_centres_on_pixel_borders(tsdf, z, shift):
    """A camera for which whole planes of voxel centres project exactly onto
    the borders between pixels (dyadic sizes: the projection is exact), each
    pixel with its own depth: the oracle's pixel in every case."""
    W, H, vs = 97, 61, z / 128
    K = Intrinsics(64.0, 64.0, 48.0 + shift, 30.0 + shift, W, H)
    rng = np.random.default_rng(int(8 * z))
    d = (z * (1 + 0.02 * rng.uniform(-1, 1, (H, W)))).astype(np.float32)
    # the camera centre is a voxel centre
    pose = np.hstack([np.eye(3), np.array([[0.5 * vs], [0.5 * vs], [0.5 * vs]])])
    origin, dims = (-128 * vs, -128 * vs, 0.0), (256, 256, 256)
    gv = tsdf.Volume(dims, vs, origin, 4.0, 1 << 13, 1 << 14, 0, 1e-4, W, H)
    ov = oracle.OracleVolume(dims, vs, origin, 4.0, capacity_blocks=1 << 13)
    coeff = 0.0015 / z
    st = ov.integrate(d, Kvec(K), pose, coeff=coeff)
    gv.integrate(torch.from_numpy(d).cuda(), K, pose, coeff=coeff)
    gst = gv.stats()
    assert st["updates"] > 20000 and gst["frame_updates"] == st["updates"]
    assert gst["frame_new_blocks"] == st["new_blocks"]
    compare_volumes(gv, ov)


@pytest.fixture(scope="module")
def gyroid():
    """Blocks of a gyroid's truncated distance, every seventh or so missing,
    and the oracle's raycast of them: brackets, stencils and empty stretches at
    every place of a block and across its borders."""
    n, vs = 96, 0.01
    q = (np.arange(n) + 0.5) * (2 * math.pi / 29.3)
    x, y, z = np.meshgrid(q, q, q, indexing="ij")
    g = np.sin(x) * np.cos(y) + np.sin(y) * np.cos(z) + np.sin(z) * np.cos(x)
    T = g / (1.2 * 2 * math.pi / 29.3) / 4.0      # about the distance in truncation widths of 4 voxels
    T[np.abs(T) > 1] = CHI
    T = T.astype(np.float32).astype(np.float64)
    ov = oracle.OracleVolume((n, n, n), vs, (0.0, 0.0, 0.0), 4.0, capacity_blocks=2048)
    rng = np.random.default_rng(3)
    for bz in range(n // 8):
        for by in range(n // 8):
            for bx in range(n // 8):
                if rng.random() < 0.15:
                    continue
                t = T[8 * bx:8 * bx + 8, 8 * by:8 * by + 8, 8 * bz:8 * bz + 8].transpose(2, 1, 0)   # x fastest
                if (t <= 1).any():
                    ov.set_block((bx, by, bz), np.ascontiguousarray(t).reshape(-1), np.full(512, 1e-3))
    K = Intrinsics(70.0, 70.0, 40.2, 29.6, 83, 59)
    pose = look_at((-0.35, 0.7, -0.25), (0.5, 0.45, 0.5))
    return n, vs, K, pose, ov.export(), ov.raycast(Kvec(K), pose, K.width, K.height, n_threads=8)


@pytest.mark.parametrize("group,dense", [(1, True), (2, False), (4, True), (8, True), (8, False), (16, False)])
def test_raycast_of_cells_at_block_borders(tsdf, gyroid, group, dense):
    n, vs, K, pose, (keys, T, P), (ov, on, flags) = gyroid
    gv = tsdf.Volume((n, n, n), vs, (0.0, 0.0, 0.0), 4.0, 2048, 4096, 0, 1e-4, K.width, K.height, dense_index=dense)
    gv.set_raycast_group(group)
    gv.import_blocks(torch.from_numpy(keys), torch.from_numpy(T).float(), torch.from_numpy(P).float())
    vert, nrm = gv.raycast(K, pose)
    torch.cuda.synchronize()
    rs = compare_raycast(vert.cpu().numpy(), nrm.cpu().numpy(), ov, on, flags, pose, vs)
    assert rs["hits"] > 1000, rs


@pytest.mark.parametrize("storage,dense,missing", [(0, True, 0.1), (0, False, 0.0), (1, True, 0.0)])
def test_mesh_of_blocks_with_several_rounds_of_triangles(tsdf, storage, dense, missing):
    """Random signs: about 1400 triangles a block, placed 512 at a time, every
    case of a cell at every place of a block; some voxels without a distance,
    some exactly zero, some neighbour blocks missing; and the same with room
    for part of the triangles, ending inside a round."""
    rng = np.random.default_rng(17 + storage)
    keys = [(x, y, z) for x in range(3) for y in range(3) for z in range(3) if rng.random() >= missing]
    T = rng.uniform(-1, 1, (len(keys), 512))
    T[rng.random(T.shape) < 0.02] = CHI
    T[rng.random(T.shape) < 0.02] = 0.0
    T = T.astype(np.float16 if storage else np.float32).astype(np.float64)
    ov, gv = load_both(tsdf, (24, 24, 24), 0.01, (-0.1, 0.0, 0.05), np.array(keys, np.int32), T, storage, dense,
                       capacity=64)
    mesh = gpu_mesh(gv)
    assert compare_meshes(mesh, ov.marching_cubes(), 0.01)["triangles"] > 20000
    n = len(mesh[0])
    cap = n - 700
    vid, t, xyz = (torch.full((cap, *s), -7, dtype=d, device="cuda")
                   for s, d in (((3,), torch.int64), ((3,), torch.float32), ((3, 3), torch.float32)))
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    gv.extract_mesh_into(vid, t, xyz, count, gv.mesh_workspace())
    torch.cuda.synchronize()
    assert int(count) == n
    for got, want in zip((vid, t, xyz), mesh):
        assert np.array_equal(got.cpu().numpy(), want[:cap])


@pytest.mark.parametrize("group,dense,close", [(1, True, False), (2, False, False), (4, True, True), (8, True, False),
                                               (8, False, True), (16, True, False)])
def test_large_frames_march_a_list_of_tiles(tsdf, gyroid, group, dense, close):
    """A ragged frame large enough to march from a list of its tiles gives
    bitwise the maps of the two half frames, which march every tile; with a
    camera that sees mostly background, and one with blocks at its plane.
    Every element is written (the maps start as NaN)."""
    n, vs, _, _, (keys, T, P), _ = gyroid
    W, H, cut = 1037, 509, 520
    gv = tsdf.Volume((n, n, n), vs, (0.0, 0.0, 0.0), 4.0, 2048, 4096, 0, 1e-4, W, H, dense_index=dense)
    gv.set_raycast_group(group)
    gv.import_blocks(torch.from_numpy(keys), torch.from_numpy(T).float(), torch.from_numpy(P).float())
    pose = look_at((0.5, 0.52, -0.02) if close else (-1.5, 2.0, -1.2), (0.5, 0.45, 0.5))
    out = {}
    for x0, x1 in ((0, W), (0, cut), (cut, W)):
        K = Intrinsics(700.0, 700.0, 500.25 - x0, 250.5, x1 - x0, H)
        maps = [torch.full((H, x1 - x0, 4), float("nan"), device="cuda") for _ in range(2)]
        gv.raycast(K, pose, *maps)
        torch.cuda.synchronize()
        out[x0, x1] = maps
    hits = int((out[0, W][0][..., 3] > 0).sum())
    assert hits > 20000
    assert close or hits < 0.9 * W * H
    for m in range(2):
        assert torch.equal(out[0, W][m], torch.cat((out[0, cut][m], out[cut, W][m]), 1))
