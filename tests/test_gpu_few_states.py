"""Evaluations of a few states (passed as a kernel argument up to 32, tiles of
fewer slices in small launches) against the oracle's sums over every voxel:
whole numbers, so equal.  The depths of the tiles are those of one slice, of
targets that end inside a tile, and of launches on either side of the rule."""

import numpy as np
import pytest

from paper_2504_19930_amd import config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 32, 33])
@pytest.mark.parametrize("score", ["dice", "ncc"])
@pytest.mark.parametrize("tshape", [(1, 9, 33), (5, 8, 32), (37, 20, 40), (70, 30, 34)])
def test_few_states_match_every_voxel(orc, score, tshape, n):
    import torch
    from paper_2504_19930_amd import binding
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rng = np.random.default_rng(11)
    top = 2 if score == "dice" else 256
    src, tgt = rng.integers(0, top, (30, 28, 36)).astype(np.uint8), rng.integers(0, top, tshape).astype(np.uint8)
    x = np.concatenate([np.deg2rad(rng.uniform(-20, 20, (n, 3))), rng.uniform(-4, 4, (n, 3))], 1)
    r = binding.Registration(dev(src), dev(tgt), config.default_params(score, 8, 1, 20.0, 4.0, seed=1))
    s, t = orc.Volume(src), orc.Volume(tgt)
    for _ in range(2):  # the second call finds the first one's sums
        got = r.evaluate(x)
        if score == "dice":
            want = np.array([orc.mask_counts(s, t, orc.recipe_words(p, s, t, nn=True)) for p in x], dtype=np.int64)
            assert np.array_equal(got[:, :want.shape[1]], want)
        else:
            want = np.array([orc.image_moments(s, t, orc.recipe_words(p, s, t, nn=False), True) for p in x],
                            dtype=np.int64)
            assert np.array_equal(got, want)
    r.close()
