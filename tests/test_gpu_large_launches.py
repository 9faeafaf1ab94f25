"""Launches of 2^24 workgroups and more, whose 2^32 threads do not fit one grid:
mask and image registrations of a flat target and many particles, single and in a
batch, evaluations of thousands of states and warps of very many frames (one
voxel each, which leaves trilinear ones to the kernel without staging)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _flat_pair(nx, nz, image):
    import torch
    rng = np.random.default_rng(4)
    src, tgt = np.zeros((48, 40, 44), np.uint8), np.zeros((nz, 1, nx), np.uint8)
    block = rng.integers(1, 256, (30, 40, 30)).astype(np.uint8)
    src[8:38, :, 7:37] = block if image else 1
    # (the volumes share their corner, 2900 voxels from the centre of rotation)
    tgt[9:37, 0, 8:36] = block[:28, 0, :28] if image else 1
    return torch.from_numpy(src).cuda(), torch.from_numpy(tgt).cuda()


def _params(score, n, seed=1):
    from paper_2504_19930_amd.config import default_params
    return dict(default_params(score, n, 1, 0.1, 3.0, seed=seed), min_overlap_frac=0.0)


def _check(r, params, picks):
    """Log-weights of the evaluated set against scores of another kernel."""
    got = r.particles()
    z = r.scores(got["states"][picks])
    assert len(np.unique(z)) > 10
    assert np.allclose(got["logw"][picks], -(1.0 - z) ** 2 * (0.5 / params["sigma_score"] ** 2), rtol=1e-12, atol=0)


def test_masks():
    from paper_2504_19930_amd.binding import Registration
    # 65536 blocks of 16^3, 64 a workgroup, x 16384 groups of particles
    src, tgt = _flat_pair(4096, 4096, False)
    p = _params("dice", 65535)
    r = Registration(src, tgt, p)
    r.run()
    _check(r, p, np.r_[0:40, 30000:30040, 65500:65535])
    r.close()


def test_images():
    import torch
    from paper_2504_19930_amd.binding import Registration
    src, tgt = _flat_pair(4096, 4096, True)
    fov = torch.ones_like(src)
    fov[:, :, 28:] = 0  # (enough to skip: by blocks; twelve a workgroup, 3076 groups)
    p = _params("ncc", 12300)
    r = Registration(src, tgt, p, src_fov=fov)
    r.run()
    got = r.particles()
    r.close()
    r = Registration(src, tgt, p, src_fov=fov)
    r.tune(layout="raw")
    r.set_particles(got["states"], 0)
    picks = np.r_[0:40, 6000:6040, 12260:12300]
    z = r.scores(got["states"][picks])
    assert len(np.unique(z)) > 10
    assert np.allclose(got["logw"][picks], -(1.0 - z) ** 2 * (0.5 / p["sigma_score"] ** 2), rtol=1e-12, atol=0)
    r.close()


def test_batch():
    from paper_2504_19930_amd.binding import Batch, Registration
    pairs = []
    for i in range(2):
        src, tgt = _flat_pair(4096, 2048, False)
        pairs.append(dict(src=src, tgt=tgt, params=dict(_params("dice", 65535, seed=i), pair_id=i)))
    b = Batch(pairs)
    b.run()
    for i, q in enumerate(pairs):
        r = Registration(q["src"], q["tgt"], q["params"])
        r.run()
        assert np.array_equal(r.particles()["logw"], b.particles(i)["logw"])
        assert len(np.unique(r.particles()["logw"])) > 10
        r.close()
    b.close()


@pytest.mark.parametrize("image", [False, True])
def test_evaluations(image):
    from paper_2504_19930_amd.binding import Registration
    # 16384 tiles x 1025 groups of states, against 820 states at a time
    src, tgt = _flat_pair(4096, 2048, image)
    r = Registration(src, tgt, _params("ncc" if image else "dice", 8))
    r.tune(tile_depth=16)
    rng = np.random.default_rng(2)
    states = rng.uniform(-1, 1, (4100, 6)) * np.array([2e-3] * 3 + [3.0] * 3)
    sums = r.evaluate(states)
    assert len(np.unique(sums[:, 1])) > 10
    assert np.array_equal(sums, np.concatenate([r.evaluate(s) for s in np.array_split(states, 5)]))
    r.close()


@pytest.mark.parametrize("interp, frames", [("nearest", 65535), ("trilinear", 16400)])
def test_warp_of_many_frames(interp, frames):
    import torch
    from paper_2504_19930_amd import binding
    src = torch.randint(1, 256, (frames, 1, 1, 1), dtype=torch.uint8, device="cuda")
    dst = torch.full((frames, 256, 512, 1), 7, dtype=torch.uint8, device="cuda")
    M = np.concatenate([np.eye(3), np.zeros((3, 1))], axis=1)
    binding.warp_apply(binding.volume(src[0]), M, interp, dst, n_frames=frames, src_frame_stride=1,
                       dst_frame_stride=256 * 512)
    assert torch.equal(dst[:, 0, 0, 0], src[:, 0, 0, 0])
    dst[:, 0, 0, 0] = 0
    for part in dst.split(8192):
        assert int(torch.count_nonzero(part)) == 0
