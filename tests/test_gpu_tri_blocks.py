"""Block launches of images with a source FOV where they are certain to be taken
(most of the source lies far from any valid sample): sums equal to the oracle's over
every voxel, at target sizes about the ends of blocks of 4^3, 8^3 and 16^3, and
with the most blocks a workgroup takes (12 for moments, 48 for histograms, whose
lists then are the longest) at the values where the 32-bit partial sums are
largest; histograms also with coordinates beyond the block test's bound."""

import numpy as np
import pytest
from scipy.ndimage import distance_transform_edt

from paper_2504_19930_amd import config

pytestmark = pytest.mark.gpu


def _fov(shape, part):
    """A ball about the volume's centre; shares of the source far from it checked."""
    z, y, x = np.meshgrid(*[np.arange(n) - 0.5 * (n - 1) for n in shape], indexing="ij")
    fov = (x ** 2 + y ** 2 + z ** 2 < (part * max(shape)) ** 2).astype(np.uint8)
    fov[shape[0] // 2, shape[1] // 2, shape[2] // 2] = 0
    away = distance_transform_edt(1 - fov)
    assert np.mean(away > 7.6) >= 0.2  # (a block of 8^3 reaches 6.1 + 1 voxels; the line is at 0.12)
    return fov


def _setup(sshape, tshape, part, kind, score, n, spacing=(1.0, 1.0, 1.0), tgt_fov=False, trans=6.0, degrees=25.0):
    import torch
    from paper_2504_19930_amd import binding
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rng = np.random.default_rng(7)
    src = rng.integers(0, 256, sshape).astype(np.uint8) if kind == "random" else np.full(sshape, kind, np.uint8)
    tgt = rng.integers(0, 256, tshape).astype(np.uint8) if kind == "random" else np.full(tshape, 255, np.uint8)
    sfov, tfov = _fov(sshape, part), None
    if tgt_fov:
        tfov = np.ones(tshape, np.uint8)
        tfov[tshape[0] // 3:tshape[0] // 2, :, tshape[2] // 4:] = 0
        tfov[0, 0, 0] = 0
    states = np.concatenate([np.deg2rad(rng.uniform(-degrees, degrees, (n, 3))), rng.uniform(-trans, trans, (n, 3))], 1)
    # the volumes' centres meet
    states[:, 3:] += 0.5 * (np.array(sshape[::-1]) * spacing - np.array(tshape[::-1]))
    states[0, :3] = 0.0
    states[1, 3:] = 500.0  # nothing overlaps
    reg = binding.Registration(dev(src), dev(tgt), dict(config.default_params(score, 8, 2, 25.0, 8.0), min_overlap_frac=0.0),
                               spacing=spacing, src_fov=dev(sfov), tgt_fov=dev(tfov), tgt_spacing=(1.0, 1.0, 1.0))
    return reg, (src, spacing, sfov), (tgt, (1.0, 1.0, 1.0), tfov), states


@pytest.mark.parametrize("tgt_fov", [False, True])
@pytest.mark.parametrize("tshape", [(2, 1, 1), (4, 17, 2), (16, 16, 16), (17, 15, 18), (18, 40, 33), (33, 35, 48),
                                    (49, 47, 52)])
def test_moments_at_the_ends_of_blocks(orc, tshape, tgt_fov):
    r, s, t, states = _setup((50, 52, 55), tshape, 0.33, "random", "ncc", 37, tgt_fov=tgt_fov)
    s, t = orc.Volume(*s), orc.Volume(*t)
    want = np.array([orc.image_moments(s, t, orc.recipe_words(p, s, t, nn=False), True) for p in states], dtype=np.int64)
    assert want[:, 0].max() > 0
    for layout in ("oct", "octtile", "lerp"):
        r.tune(layout)
        assert np.array_equal(r.evaluate(states), want), layout
    r.close()


@pytest.mark.parametrize("kind", [0, 255, "random"])
def test_moments_of_twelve_blocks_a_workgroup(orc, kind):
    # 125 blocks of 16^3 x 200 groups of particles / 2048 = 12.2
    n = 800
    r, s, t, states = _setup((110, 100, 104), (72, 72, 72), 0.33, kind, "ncc", n, trans=3.0)
    s, t = orc.Volume(*s), orc.Volume(*t)
    picks = np.r_[0:12, 398:404, n - 8:n]
    want = np.array([orc.image_moments(s, t, orc.recipe_words(p, s, t, nn=False), True) for p in states[picks]],
                    dtype=np.int64)
    assert want[:, 0].max() > 100000
    for layout in ("oct", "octtile", "lerp"):
        r.tune(layout)
        assert np.array_equal(r.evaluate(states)[picks], want), layout
    r.close()


def test_moments_of_voxels_valid_throughout(orc):
    # whole blocks of 16^3 by the hundred: every lane takes 192 samples and more
    n = 800
    r, s, t, states = _setup((128, 130, 126), (72, 72, 72), 0.40, 0, "ssd", n, trans=1.0, degrees=2.0)
    s, t = orc.Volume(*s), orc.Volume(*t)
    picks = np.r_[0, 2:10, n - 4:n]
    want = np.array([orc.image_moments(s, t, orc.recipe_words(p, s, t, nn=False), True) for p in states[picks]],
                    dtype=np.int64)
    for layout in ("oct", "octtile", "lerp"):
        r.tune(layout)
        assert np.array_equal(r.evaluate(states)[picks], want), layout
    r.close()


@pytest.mark.parametrize("tshape, n, spacing, trans", [
    ((5, 6, 7), 21, (1.0, 1.0, 1.0), 4.0),
    ((34, 31, 33), 40, (1.0, 1.0, 1.0), 6.0),
    ((80, 90, 100), 1900, (1.0, 1.0, 1.0), 5.0),    # 210 blocks x 475 groups / 2048 = 48.7
    ((24, 24, 24), 30, (1e-5, 1.0, 1.0), 4.0),      # coordinates of 10^6
])
def test_histograms(orc, tshape, n, spacing, trans):
    sshape = (70, 72, 75) if min(tshape) < 80 else (120, 124, 118)
    r, s, t, states = _setup(sshape, tshape, 0.33, "random", "mi", n, spacing=spacing, trans=trans)
    if spacing[0] < 1.0:
        states[2:, 3] = np.random.default_rng(1).uniform(-2e-4, 8e-4, n - 2)
        states[2:, 1:3] = np.random.default_rng(2).uniform(-2e-6, 2e-6, (n - 2, 2))
        states[0, 3] = 3e-4
    s, t = orc.Volume(*s), orc.Volume(*t)
    picks = np.unique(np.r_[0:min(n, 14), max(0, n - 12):n])
    want = np.array([orc.mi_score(orc.joint_histogram(s, t, orc.recipe_words(p, s, t, nn=False))) for p in states[picks]])
    assert len(np.unique(want)) > 3
    for layout in ("oct", "octtile", "lerp"):
        r.tune(layout)
        assert np.array_equal(r.scores(states)[picks], want), layout
    r.close()
