"""warp_apply at views far apart, where the target's x axis falls on the source's
z axis: the box of a tile hardly shrinks with its depth, so small launches, which
prefer shallow tiles, have to keep the depth whose box fits the LDS.  Bytes equal
to the oracle's."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("interp", [0, 1])
@pytest.mark.parametrize("shape, degrees, frames, spacing", [
    ((131, 117, 95), (-20, 90, 5), 1, (1.0, 1.0, 1.0)),
    ((131, 117, 95), (-20, -90, 5), 3, (1.0, 1.0, 1.0)),
    ((131, 117, 95), (10, 90, 170), 1, (1.0, 1.0, 1.0)),
    ((131, 117, 95), (12, 86, 176), 2, (1.0, 1.0, 1.0)),
    ((131, 117, 95), (-20, 85, 0), 1, (1.0, 1.0, 1.0)),
    ((97, 89, 71), (10, 80, 10), 1, (1.0, 1.0, 1.0)),
    ((64, 64, 64), (10, 80, 10), 1, (1.0, 1.0, 1.0)),
    ((64, 60, 50), (5, 75, -8), 1, (0.9, 1.0, 1.1)),
])
def test_views_match_the_oracle(orc, interp, shape, degrees, frames, spacing):
    import torch
    from paper_2504_19930_amd import binding
    rng = np.random.default_rng(9)
    src = rng.integers(0, 256, (frames,) + shape[::-1]).astype(np.uint8)
    p = np.concatenate([np.deg2rad(degrees), [1.3, -0.7, 0.4]])
    M = orc.phys_matrix(p, shape, spacing)
    s = torch.from_numpy(src).cuda()
    dst = torch.full(src.shape, 7, dtype=torch.uint8, device="cuda")
    size = int(np.prod(shape))
    binding.warp_apply(binding.volume(s[0], spacing), M, "trilinear" if interp else "nearest", dst, spacing=spacing,
                       n_frames=frames, src_frame_stride=size, dst_frame_stride=size)
    torch.cuda.synchronize()
    got = dst.cpu().numpy()
    for f in range(frames):
        ref = orc.warp_apply(orc.Volume(src[f], spacing), M, bool(interp), shape, spacing)
        assert np.array_equal(got[f], ref), f
