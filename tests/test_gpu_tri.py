"""Trilinear sums of the one-gather layouts (blocks of the target decided by
the field of the valid source cells) against the oracle's sums over every
voxel: whole numbers, so equal.  Sizes where the blocks of 4^3, 8^3 and 16^3
end, flat volumes (no certainly valid cell), FOVs of both volumes, transforms
in, across and outside the source, coordinates beyond the block test's bound,
and the values at which the 32-bit partial sums are largest."""

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


CASES = [
    ((1, 1, 1), (1, 1, 1), None, (1.0, 1.0, 1.0), 0.5, "random"),
    ((5, 3, 33), (4, 17, 2), None, (1.0, 1.0, 1.0), 3.0, "random"),
    ((1, 40, 40), (18, 40, 33), "src", (1.0, 1.0, 1.0), 3.0, "random"),
    ((34, 31, 32), (33, 35, 48), "both", (1.0, 1.0, 1.0), 5.0, "random"),
    ((52, 51, 65), (49, 47, 52), None, (1.0, 1.0, 1.0), 8.0, "random"),
    ((48, 48, 52), (41, 44, 50), "src", (0.6, 1.2, 0.8), 8.0, "random"),
    ((24, 24, 24), (24, 24, 24), None, (1e-5, 1.0, 1.0), 4.0, "random"),
    ((80, 80, 80), (72, 72, 72), None, (1.0, 1.0, 1.0), 2.0, "extreme"),
    ((80, 80, 80), (72, 72, 72), "both", (1.0, 1.0, 1.0), 2.0, "extreme"),
]


@pytest.mark.parametrize("sshape, tshape, fov, spacing, trans, kind", CASES)
def test_one_gather_sums_match_every_voxel(smc, orc, sshape, tshape, fov, spacing, trans, kind):
    import torch
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rng = np.random.default_rng(7)
    if kind == "extreme":
        src, tgt = np.zeros(sshape, np.uint8), np.full(tshape, 255, np.uint8)
    else:
        src = rng.integers(0, 256, sshape).astype(np.uint8)
        tgt = rng.integers(0, 256, tshape).astype(np.uint8)
    z, y, x = np.meshgrid(*[np.linspace(-1, 1, n) if n > 1 else np.zeros(1) for n in sshape], indexing="ij")
    sfov = ((x ** 2 + y ** 2 + 0.5 * z ** 2) < 1.1).astype(np.uint8) if fov else None
    tfov = None
    if fov == "both":
        tfov = np.ones(tshape, np.uint8)
        tfov[5:11, :, 3:] = 0
    n = 37
    states = np.concatenate([np.deg2rad(rng.uniform(-25, 25, (n, 3))), rng.uniform(-trans, trans, (n, 3))], 1)
    states[0] = 0.0
    states[1, 3:] = 500.0  # nothing overlaps
    prm = config.default_params("ncc", n, 2, 25.0, 8.0, seed=3)
    r = smc.Registration(dev(src), dev(tgt), prm, spacing=spacing, src_fov=dev(sfov), tgt_fov=dev(tfov),
                         tgt_spacing=(1.0, 1.0, 1.0))
    s, t = orc.Volume(src, spacing, sfov), orc.Volume(tgt, (1.0, 1.0, 1.0), tfov)
    want = np.array([orc.image_moments(s, t, orc.recipe_words(p, s, t, nn=False), True) for p in states], dtype=np.int64)
    for layout in ("oct", "octtile", "lerp"):
        r.tune(layout)
        assert np.array_equal(r.evaluate(states), want), layout
    r.close()
