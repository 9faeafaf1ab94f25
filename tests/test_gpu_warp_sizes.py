"""warp_apply over odd sizes, views at odd addresses and rotations that reach
each depth of the staged tiles (16, 8, 4 slices) and the direct kernel, with the
numbers of frames on either side of a workgroup's group: bytes equal to the
oracle's.  Sources from 16 bytes on, whose last 16-byte chunks end past the
volume."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rotation(angle):
    c, s = np.cos(angle), np.sin(angle)
    rx = np.array([[1, 0, 0], [0, c, -s], [0, s, c]])
    ry = np.array([[c, 0, s], [0, 1, 0], [-s, 0, c]])
    rz = np.array([[c, -s, 0], [s, c, 0], [0, 0, 1]])
    return rz @ rx @ ry


@pytest.mark.parametrize("interp", [0, 1])
@pytest.mark.parametrize("sshape, tshape, angle, scale, frames, offset", [
    ((1, 1, 16), (1, 1, 16), 0.0, 1.0, 1, 0),
    ((1, 3, 7), (2, 5, 9), 5.0, 1.0, 3, 1),
    ((9, 10, 33), (12, 11, 35), 3.0, 1.0, 5, 3),
    ((21, 34, 51), (23, 35, 49), 12.0, 1.0, 4, 0),
    ((40, 37, 45), (41, 40, 47), 20.0, 1.0, 2, 2),
    ((48, 50, 63), (45, 52, 61), 27.0, 1.0, 9, 1),
    ((48, 50, 63), (45, 52, 61), 33.0, 1.25, 3, 0),
    ((60, 61, 62), (30, 31, 33), 25.0, 2.5, 2, 5),   # no box fits: direct
    ((40, 128, 132), (40, 130, 134), 10.0, 1.0, 6, 1),
])
def test_warp_matches_the_oracle(orc, interp, sshape, tshape, angle, scale, frames, offset):
    import torch
    from paper_2504_19930_amd import binding
    rng = np.random.default_rng(8)
    src = rng.integers(0, 256, (frames,) + sshape).astype(np.uint8)
    size, out_size = int(np.prod(sshape)), int(np.prod(tshape))
    flat = torch.zeros(frames * size + offset, dtype=torch.uint8, device="cuda")
    s = flat[offset:].view(src.shape)
    s.copy_(torch.from_numpy(src))
    out = torch.full((frames * out_size + offset + 64,), 7, dtype=torch.uint8, device="cuda")
    dst = out[offset:offset + frames * out_size].view((frames,) + tshape)
    R = scale * _rotation(np.deg2rad(angle))
    cs, ct = [0.5 * (np.array(q[::-1]) - 1.0) for q in (sshape, tshape)]
    M = np.concatenate([R, (cs - R @ ct + 0.3)[:, None]], axis=1)
    mode = "trilinear" if interp else "nearest"
    binding.warp_apply(binding.volume(s[0]), M, mode, dst, n_frames=frames, src_frame_stride=size,
                       dst_frame_stride=out_size)
    torch.cuda.synchronize()
    got = dst.cpu().numpy()
    for f in range(frames):
        assert np.array_equal(got[f], orc.warp_apply(orc.Volume(src[f]), M, bool(interp), tshape[::-1])), f
    edge = out.cpu().numpy()
    assert (edge[:offset] == 7).all() and (edge[offset + frames * out_size:] == 7).all()
