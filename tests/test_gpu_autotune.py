"""smc_autotune leaves the particles per group and the tile depth alone where the
launches that it times use neither -- masks, and the one-gather layouts of a
source with a FOV: what differed between such candidates was noise, and
smc_evaluate, which uses them, would run with what noise picked."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _params(score, n):
    from paper_2504_19930_amd.config import default_params
    return default_params(score, n, 3, 15.0, 6.0, seed=4)


def _pair(shape, seed):
    import torch
    z, y, x = np.meshgrid(*[np.arange(n) - 0.5 * (n - 1) for n in shape[::-1]], indexing="ij")
    r = (x / shape[0]) ** 2 + (y / shape[1]) ** 2 + (z / shape[2]) ** 2
    rng = np.random.default_rng(seed)
    img = np.clip(200 * np.exp(-12 * r) + rng.integers(0, 40, r.shape), 0, 255).astype(np.uint8)
    return torch.from_numpy(img).cuda(), torch.from_numpy((r < 0.08).astype(np.uint8)).cuda()


@pytest.mark.parametrize("n", [40, 50, 60, 70, 80, 90])
@pytest.mark.parametrize("own", [(4, 16), (16, 40)])
def test_masks_keep_their_settings(n, own):
    from paper_2504_19930_amd.binding import Registration
    _, mask = _pair((41, 38, 36), n)
    reg = Registration(mask, mask, _params("dice", n))
    reg.tune(particles_per_group=own[0], tile_depth=own[1])
    t = reg.autotune(1)
    assert (t["particles_per_group"], t["tile_depth"]) == own and t["ms"] > 0.0
    reg.close()


@pytest.mark.parametrize("score", ["ncc", "mi"])
@pytest.mark.parametrize("n", [41, 51, 61, 71])
def test_images_with_a_fov_keep_them_in_one_gather_layouts(score, n):
    from paper_2504_19930_amd.binding import Registration
    img, _ = _pair((41, 38, 36), n)
    fov = img.new_ones(img.shape)
    fov[:, :, 24:] = 0  # (enough to skip: the one-gather layouts go by blocks)
    reg = Registration(img, img, _params(score, n), src_fov=fov)
    reg.tune(particles_per_group=16, tile_depth=40)
    t = reg.autotune(1)
    if t["layout"] >= 3:
        assert (t["particles_per_group"], t["tile_depth"]) == (16, 40)
    reg.close()
