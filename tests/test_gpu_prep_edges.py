"""Preparation in rounds (frames whose pixels are wider than blocks) together with
the learned variance, the batched steps and a full candidate list (needs an
MI355X)."""

import numpy as np
import pytest
import torch

from synthetic.configs import sequence_frame, small_orbit
from tests.parity import gpu_volume_for
from tests.test_gpu_batch import STAT_KEYS, sorted_export

pytestmark = pytest.mark.gpu

SIZES = ((60, 45), (24, 18), (13, 9))


@pytest.fixture(scope="module")
def tsdf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_7194_amd as m

    m.lib()
    return m


def wide(size):
    return small_orbit(width=size[0], height=size[1], n_frames=2, G=512, vs=0.004)


def mlp_params():
    from paper_1311_7194_amd import mlp as M

    return M.params_from_values(M.init_params(3))


@pytest.mark.parametrize("size", SIZES)
def test_rounds_with_the_learned_variance(tsdf, size):
    """The learned variance shares its LDS with the block lists.  The blocks of a
    frame and, on the first one, the distances do not depend on the variance."""
    spec = wide(size)
    a, b = gpu_volume_for(spec), gpu_volume_for(spec)
    d, p = sequence_frame(spec, 0)
    a.integrate(d.cuda(), spec.K, p)
    b.integrate(d.cuda(), spec.K, p, tsdf.NOISE_MLP, 0.0015, mlp_params())
    sa, sb = a.stats(), b.stats()
    assert all(sa[k] == sb[k] for k in STAT_KEYS) and sa["status_flags"] == 0
    ka, ta, _ = sorted_export(a)
    kb, tb, _ = sorted_export(b)
    assert np.array_equal(ka, kb) and torch.equal(ta, tb) and len(ka) > 400


@pytest.mark.parametrize("noise,graph,persistent", [("quadratic", True, False), ("mlp", False, False),
                                                    ("quadratic", False, True), ("mlp", False, True)])
def test_rounds_in_a_batch(tsdf, noise, graph, persistent):
    """Scenes that take several rounds a tile, one that takes one, and one that
    sits out the second step: volumes and maps are those of the single calls."""
    specs = [wide(s) for s in SIZES] + [small_orbit(width=80, height=60, n_frames=2, G=256, vs=0.008, seed=2)]
    kind, params = (tsdf.NOISE_MLP, mlp_params()) if noise == "mlp" else (tsdf.NOISE_QUADRATIC, None)
    batched, plain = [gpu_volume_for(s) for s in specs], [gpu_volume_for(s) for s in specs]
    b = tsdf.Batch(batched, [s.K for s in specs], graph=graph)
    b.set_persistent(persistent)
    for t in range(2):
        frames = [sequence_frame(s, t) for s in specs]
        out = [t == 1 and k == 1 for k in range(len(specs))]
        depths = [None if o else d.cuda().contiguous() for (d, _), o in zip(frames, out)]
        b.step(depths, [None if o else p for (_, p), o in zip(frames, out)], kind, 0.0015, params)
        for k, s in enumerate(specs):
            if out[k]:
                continue
            plain[k].integrate(depths[k], s.K, frames[k][1], kind, 0.0015, params)
            vert, nrm = plain[k].raycast(s.K, frames[k][1])
            torch.cuda.synchronize()
            assert torch.equal(vert, b.vertex[k]) and torch.equal(nrm, b.normal[k]), (t, k)
    for k in range(len(specs)):
        sb, sp = batched[k].stats(), plain[k].stats()
        assert all(sb[key] == sp[key] for key in STAT_KEYS) and sb["status_flags"] == 0, k
        for x, y in zip(sorted_export(batched[k]), sorted_export(plain[k])):
            assert np.array_equal(np.asarray(x), np.asarray(y)), k


@pytest.mark.parametrize("cand", [1, 100, 1500])
def test_rounds_with_a_full_candidate_list(tsdf, cand):
    """A frame with more blocks than the candidate list holds, several rounds of
    them per tile: that flag alone is raised, and the frame after it finds all of
    its own blocks (no mark of a block that was turned away is left)."""
    spec = wide((24, 18))
    K = spec.K
    g = spec.grid
    gv = tsdf.Volume(g.dims, g.voxel_size, g.origin, g.trunc_voxels, g.capacity_blocks, g.hash_slots, 0, 1e-4, K.width,
                     K.height, max_candidates=cand)
    ref = gpu_volume_for(spec)
    d, p = sequence_frame(spec, 0)
    one = torch.zeros_like(d)
    j, i = K.height // 2, K.width // 2   # (the orbit looks at the grid's middle)
    one[j, i] = d[j, i]
    ref.integrate(one.cuda(), K, p)
    want = ref.stats()
    assert want["frame_candidates"] > 0
    gv.integrate(d.cuda(), K, p)
    gv.integrate(one.cuda(), K, p)
    got = gv.stats()
    assert got["status_flags"] == tsdf.tsdf.FLAG_CAND_FULL
    if want["frame_candidates"] <= cand:
        assert got["frame_candidates"] == want["frame_candidates"]
        assert got["frame_updates"] == want["frame_updates"]
        assert got["frame_touched_blocks"] == want["frame_touched_blocks"]
    else:
        assert got["frame_candidates"] >= want["frame_candidates"]
