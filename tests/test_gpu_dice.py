"""The filter's mask launches (blocks of the target decided by the source's
distance field) against the oracle's counts of every voxel, at the sizes
where the blocks of 4^3, 8^3 and 16^3 and the 32-voxel bitmap words end, and
for transforms that put the source in, across and far outside the target.
One iteration's log-weights come from whole counts, so they are compared at
the last bits of one FP64 formula (1e-12 relative)."""

import numpy as np
import pytest

from paper_2504_19930_amd import config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19930_amd import binding
    binding.lib()
    return binding


def _mask(shape, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "full":
        return np.ones(shape, np.uint8)
    if kind == "sparse":
        return (rng.random(shape) < 0.01).astype(np.uint8)
    z, y, x = np.meshgrid(*[np.arange(n) - 0.5 * (n - 1) for n in shape], indexing="ij")
    r = (x / (0.45 * shape[2])) ** 2 + (y / (0.4 * shape[1])) ** 2 + (z / (0.4 * shape[0])) ** 2
    return (r <= 1.0).astype(np.uint8)


@pytest.mark.parametrize("kind", ["full", "ball", "sparse"])
@pytest.mark.parametrize("sshape, tshape, fov, spacing, trans", [
    ((1, 1, 1), (1, 1, 1), False, (1.0, 1.0, 1.0), 1.0),
    ((5, 3, 33), (4, 17, 2), False, (1.0, 1.0, 1.0), 3.0),
    ((16, 31, 32), (33, 16, 8), True, (1.0, 1.0, 1.0), 6.0),
    ((40, 37, 65), (49, 47, 52), False, (1.0, 1.0, 1.0), 8.0),
    ((40, 48, 44), (41, 44, 50), True, (0.5, 1.3, 0.8), 8.0),     # anisotropic: the image of a block is no cube
    ((24, 24, 24), (24, 24, 24), False, (1e-5, 1.0, 1.0), 4.0),   # coordinates beyond the block test's bound
])
def test_dice_launch_counts_match_every_voxel(smc, orc, kind, sshape, tshape, fov, spacing, trans):
    import torch
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    src, tgt = _mask(sshape, kind, 1), _mask(tshape, kind, 2)
    sfov = (np.random.default_rng(3).random(sshape) < 0.9).astype(np.uint8) if fov else None
    tfov = np.ones(tshape, np.uint8) if fov else None
    if fov:
        tfov[:, : tshape[1] // 2, 3:9] = 0
    prm = config.default_params("dice", 70, 1, 25.0, trans, seed=5)
    r = smc.Registration(dev(src), dev(tgt), prm, spacing=spacing, src_fov=dev(sfov) if fov else None,
                         tgt_fov=dev(tfov) if fov else None, tgt_spacing=(1.0, 1.0, 1.0))
    x = r.particles()["states"]
    r.run()
    got = r.particles()["logw"]
    s, t = orc.Volume(src, spacing, sfov), orc.Volume(tgt, (1.0, 1.0, 1.0), tfov)
    counts = np.array([orc.mask_counts(s, t, orc.recipe_words(p, s, t, nn=True)) for p in x], dtype=np.int64)
    t_on = int((tgt * (tfov if fov else 1)).sum())
    den = counts[:, 1] + t_on
    z = np.where(den > 0, 2.0 * counts[:, 2] / np.maximum(den, 1), 0.0)
    want = -((1.0 - z) ** 2) * (0.5 / prm["sigma_score"] ** 2)
    assert np.allclose(got, want, rtol=1e-12, atol=0.0)
    w = r.profile_work()
    assert w["interior"] <= w["evaluated"] <= w["covered"] == tgt.size * 72  # 70 particles, the estimate twice
    r.close()
