"""The raycast where its shortcuts could show: the refinement inside a cell, rays
with many brackets that are none, marches from a tile list (needs an MI355X)."""

import numpy as np
import pytest
import torch

from synthetic import Intrinsics, look_at

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tsdf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_7194_amd as m

    m.lib()
    return m


def trilinear(T, q, dtype):
    """F at the points q of a grid, every interpolation rounded once to dtype."""
    c = np.minimum(np.floor(q).astype(int), np.array(T.shape) - 2)
    fr = (q - c).astype(dtype)

    def lerp(a, b, t):
        return (a.astype(np.float64) + t.astype(np.float64) * (b - a).astype(dtype)).astype(dtype)

    v = {k: T[c[:, 0] + (k & 1), c[:, 1] + (k >> 1 & 1), c[:, 2] + (k >> 2)].astype(dtype) for k in range(8)}
    x = [lerp(v[k], v[k + 1], fr[:, 0]) for k in (0, 2, 4, 6)]
    return lerp(lerp(x[0], x[1], fr[:, 1]), lerp(x[2], x[3], fr[:, 1]), fr[:, 2])


def sampled_search(T, o, d):
    """Crossings of the rays o + s d (voxel-centre coordinates) as tsdf_raycast
    defines them, every point evaluated from the voxels in single precision."""
    n, h, last = len(d), 0.5, len(T) - 1
    lo, prev = np.full(n, np.nan), np.full(n, np.nan)
    for k in range(1, 160):
        q = o + k * h * d
        ok = ((q >= 0) & (q < last)).all(1)
        F = np.full(n, np.nan)
        F[ok] = trilinear(T, q[ok], np.float32)
        lo[np.isnan(lo) & (prev > 0) & (F <= 0)] = (k - 1) * h
        prev = F
    hit = ~np.isnan(lo)
    d, a = d[hit], lo[hit]
    b = a + h
    at = lambda s: trilinear(T, o + s[:, None] * d, np.float32)   # noqa: E731
    Fa, Fb = at(a), at(b)
    for _ in range(6):
        p = [at(a + (b - a) * (m + 1) * 0.25) for m in range(3)]
        k = np.where(p[0] <= 0, 0, np.where(p[1] <= 0, 1, np.where(p[2] <= 0, 2, 3)))
        w = (b - a) * 0.25
        Fa, Fb = np.choose(k, [Fa] + p), np.choose(k, p + [Fb])
        a = a + w * k
        b = a + w
    return hit, a + (b - a) * (Fa.astype(np.float64) / (Fa.astype(np.float64) - Fb))


def rays(K, pose):
    j, i = np.meshgrid(np.arange(K.height), np.arange(K.width), indexing="ij")
    d = np.stack([(i - K.cx) / K.fx, (j - K.cy) / K.fy, np.ones(i.shape)], -1).reshape(-1, 3) @ pose[:, :3].T
    return d / np.linalg.norm(d, axis=1, keepdims=True)


@pytest.mark.parametrize("group,dense", [(1, True), (4, False), (8, True)])
def test_refinement_is_the_search_over_sampled_points(tsdf, group, dense):
    """Strongly curved cells around the world's origin, where a vertex is stored
    to 6e-8 voxel: the crossings are those of the search over sampled points,
    within that rounding (1.2e-7 along a ray) but for the rays whose root lies
    so near a point that the sign there is rounding (under one in a hundred),
    and |F| at them is no larger than at the search's own."""
    W = H = 64
    K = Intrinsics(360.0, 360.0, W / 2.0, H / 2.0, W, H)
    gv = tsdf.Volume((8, 8, 8), 1.0, (-4.0, -4.0, -4.0), 4.0, 4, 8, 0, 1e-4, W, H, dense_index=dense)
    gv.set_raycast_group(group)
    c = np.arange(8) - 3.5
    x, y, z = np.meshgrid(c, c, c, indexing="ij")
    inner = (np.abs(x) < 2) & (np.abs(y) < 2) & (np.abs(z) < 2)
    err, res, ref = [], [], []
    for seed in range(16):
        rng = np.random.default_rng(seed)
        T = rng.uniform(0.2, 0.9, (8, 8, 8))
        T[inner] = rng.uniform(-0.9, 0.9, inner.sum())
        T = T.astype(np.float32)
        gv.import_blocks(torch.zeros((1, 3), dtype=torch.int32),
                         torch.from_numpy(np.ascontiguousarray(T.transpose(2, 1, 0))).reshape(1, 512),
                         torch.full((1, 512), 1e-3))
        pose = look_at(np.array([-8.0, 9.0, -10.0]) + rng.normal(size=3), (0.0, 0.0, 0.0))
        vert, _ = gv.raycast(K, pose)
        torch.cuda.synchronize()
        vert = vert.cpu().numpy().reshape(-1, 4)
        d = rays(K, pose)
        hit, s = sampled_search(T, pose[:, 3] + 3.5, d)
        want = np.full((W * H, 3), np.nan)
        want[hit] = pose[:, 3] + s[:, None] * d[hit]
        both = (vert[:, 3] > 0) & hit & (np.abs(want) < 1.4).all(1)
        err.append(np.linalg.norm(vert[both, :3] - want[both], axis=1))
        res.append(np.abs(trilinear(T, vert[both, :3] + 3.5, np.float64)))
        ref.append(np.abs(trilinear(T, want[both].astype(np.float32) + 3.5, np.float64)))
    err, res, ref = (np.concatenate(v) for v in (err, res, ref))
    print(f"[raycast] {len(err)} crossings, {np.mean(err > 1.2e-7):.4f} further than 1.2e-7 voxel from the search's; "
          f"mean |F| {res.mean():.3e}, at the search's {ref.mean():.3e}", flush=True)
    assert len(err) > 5000
    assert np.mean(err > 1.2e-7) <= 0.01
    assert res.mean() <= 1.02 * ref.mean()


def test_candidates_without_a_crossing(tsdf):
    """Voxels of random values, one in twenty below zero: most steps of a ray
    see cells where a bracket can begin and end, few of them have a crossing.
    Every group size finds the crossings of the search over all samples and
    gives bitwise the same maps (coordinates up to 16: rounding 1e-6 apart)."""
    n, W, H = 32, 96, 80
    K = Intrinsics(150.0, 150.0, 47.3, 39.6, W, H)
    rng = np.random.default_rng(11)
    T = rng.uniform(0.05, 0.95, (n, n, n)).astype(np.float32)
    T[rng.random(T.shape) < 0.05] *= -1
    gv = tsdf.Volume((n, n, n), 1.0, (-16.0, -16.0, -16.0), 4.0, 64, 128, 0, 1e-4, W, H)
    m = n // 8
    keys = [(x, y, z) for x in range(m) for y in range(m) for z in range(m)]
    blocks = [T[8 * x:8 * x + 8, 8 * y:8 * y + 8, 8 * z:8 * z + 8].transpose(2, 1, 0).reshape(-1) for x, y, z in keys]
    gv.import_blocks(torch.tensor(keys, dtype=torch.int32), torch.from_numpy(np.stack(blocks)),
                     torch.full((len(keys), 512), 1e-3))
    pose = look_at((-38.0, 21.0, -25.0), (0.0, 0.0, 0.0))
    d = rays(K, pose)
    hit, s = sampled_search(T, pose[:, 3] + 15.5, d)
    want = pose[:, 3] + s[:, None] * d[hit]
    inner = (np.abs(want) < 14.4).all(1)   # every sample of the normal in the grid
    maps = []
    for group in (1, 2, 4, 8, 16):
        gv.set_raycast_group(group)
        maps.append([t.cpu().numpy().reshape(-1, 4) for t in gv.raycast(K, pose)])
        assert np.array_equal(maps[0][0], maps[-1][0]) and np.array_equal(maps[0][1], maps[-1][1]), group
    vert = maps[0][0]
    got = vert[hit, 3] > 0
    assert inner.sum() > 3000 and not (vert[~hit, 3] > 0).any()
    assert np.mean(got[inner]) > 0.999
    assert np.linalg.norm(vert[hit, :3] - want, axis=1)[got].max() < 1e-4   # a bracket of the search
    assert np.mean(np.linalg.norm(vert[hit, :3] - want, axis=1)[got] < 4e-6) > 0.99


@pytest.fixture(scope="module")
def shells():
    """Blocks of a sphere and a plane inside a 128^3 grid, half-precision values."""
    n = 128
    q = np.arange(n) + 0.5
    x, y, z = np.meshgrid(q, q, q, indexing="ij")
    T = np.minimum(np.sqrt((x - 64) ** 2 + (y - 64) ** 2 + (z - 64) ** 2) - 40, y - 10) / 4
    T[np.abs(T) > 1] = 2.0
    T = T.astype(np.float16)
    keys, blocks = [], []
    for k in np.ndindex(n // 8, n // 8, n // 8):
        t = T[tuple(slice(8 * a, 8 * a + 8) for a in k)]
        if (t <= 1).any():
            keys.append(k)
            blocks.append(t.transpose(2, 1, 0).reshape(-1))
    return n, torch.tensor(keys, dtype=torch.int32), torch.from_numpy(np.stack(blocks))


def shells_volume(tsdf, shells, storage, dense, W, H):
    n, keys, T = shells
    gv = tsdf.Volume((n, n, n), 0.01, (0.0, 0.0, 0.0), 4.0, 4096, 8192, storage, 1e-4, W, H, dense_index=dense)
    gv.import_blocks(keys, T.to(gv.elem_dtype), torch.full(T.shape, 1e-3))
    return gv


@pytest.mark.parametrize("group,dense", [(1, False), (2, True), (8, True), (16, False)])
def test_half_precision_from_a_tile_list(tsdf, shells, group, dense):
    """A ragged half-precision frame of 8320 tiles against its two halves, which
    march every tile: bitwise the same."""
    W, H, cut = 1037, 509, 520
    gv = shells_volume(tsdf, shells, 1, dense, W, H)
    gv.set_raycast_group(group)
    pose = look_at((-0.9, 1.6, -1.1), (0.6, 0.5, 0.6))
    out = {}
    for x0, x1 in ((0, W), (0, cut), (cut, W)):
        maps = [torch.full((H, x1 - x0, 4), float("nan"), device="cuda") for _ in range(2)]
        gv.raycast(Intrinsics(700.0, 700.0, 500.25 - x0, 250.5, x1 - x0, H), pose, *maps)
        torch.cuda.synchronize()
        out[x0, x1] = maps
    hits = int((out[0, W][0][..., 3] > 0).sum())
    assert 20000 < hits < 0.9 * W * H
    for m in range(2):
        assert torch.equal(out[0, W][m], torch.cat((out[0, cut][m], out[cut, W][m]), 1))


@pytest.mark.parametrize("W,H", [(120, 90), (512, 255), (512, 256), (801, 650), (1040, 512)])
@pytest.mark.parametrize("storage", [0, 1])
def test_autotuned_form_gives_the_same_maps(tsdf, shells, W, H, storage):
    """Frames below and above the sizes from which the list is timed (2048 tiles)
    and taken untuned (8192): whatever the autotuner keeps, the maps of that frame
    and of smaller and larger ones are bitwise those before."""
    gv = shells_volume(tsdf, shells, storage, True, 1100, 700)
    pose = look_at((-0.9, 1.6, -1.1), (0.6, 0.5, 0.6))
    Ks = [Intrinsics(0.7 * w, 0.7 * w, 0.48 * w, 0.49 * h, w, h) for w, h in ((W, H), (160, 120), (1100, 700))]
    before = [gv.raycast(K, pose) for K in Ks]
    group, ms = gv.autotune_raycast(Ks[0], pose)
    assert group in (1, 2, 4, 8, 16) and gv.raycast_group == group and ms > 0
    for K, maps in zip(Ks, before):
        assert int((maps[0][..., 3] > 0).sum()) > 1000
        after = [torch.full_like(m, float("nan")) for m in maps]
        gv.raycast(K, pose, *after)
        assert all(torch.equal(a, b) for a, b in zip(maps, after))


@pytest.mark.parametrize("group,storage,dense", [(1, 0, True), (8, 0, False), (16, 1, True)])
def test_footprint_counts_the_blocks_of_all_samples(tsdf, shells, group, storage, dense):
    """The count holds every block that a valid sample up to a ray's crossing is
    based in, not those of the samples around the crossing alone, and none
    but allocated blocks with a sample up to the crossing's step."""
    W, H = 160, 120
    n, keys, blocks = shells
    gv = shells_volume(tsdf, shells, storage, dense, W, H)
    gv.set_raycast_group(group)
    T = np.full((n, n, n), 2.0, np.float32)
    allocated = np.zeros((n // 8,) * 3, bool)
    for k, b in zip(keys.tolist(), blocks.float().numpy()):
        T[tuple(slice(8 * a, 8 * a + 8) for a in k)] = b.reshape(8, 8, 8).transpose(2, 1, 0)
        allocated[tuple(k)] = True
    K = Intrinsics(112.0, 112.0, 76.8, 58.8, W, H)
    pose = look_at((-0.9, 1.6, -1.1), (0.6, 0.5, 0.6))
    d = rays(K, pose)
    q0 = pose[:, 3] / 0.01 - 0.5
    chi = T > 1
    need, may = np.zeros_like(allocated), np.zeros_like(allocated)
    prev, over = np.full(W * H, np.nan), np.zeros(W * H, int)   # over: samples past the crossing
    for s in range(1, 900):
        live = over < group
        q = q0 + 0.5 * s * d
        live &= ((q >= 0) & (q < n - 1)).all(1)
        c = np.floor(q[live]).astype(int)
        B = tuple((c >> 3).T)
        may[B] |= allocated[B]
        ok = ~np.any([chi[c[:, 0] + (e & 1), c[:, 1] + (e >> 1 & 1), c[:, 2] + (e >> 2)] for e in range(8)], axis=0)
        F = np.full(W * H, np.nan)
        F[live] = np.where(ok, trilinear(T, q[live], np.float32), np.nan)
        first = ok & (over[live] == 0)
        need[tuple((c[first] >> 3).T)] = True
        over += (over > 0) | ((prev > 0) & (F <= 0))
        prev = F
    count, vert, _ = gv.raycast_footprint(K, pose)
    print(f"[raycast] footprint {count} blocks, {need.sum()} with a valid sample, {may.sum()} with any", flush=True)
    assert int((vert[..., 3] > 0).sum()) > 1000
    assert need.sum() - 1 <= count <= may.sum() + 1   # (a sample within rounding of a border)
    assert need.sum() > 300
