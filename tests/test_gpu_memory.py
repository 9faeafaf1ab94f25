"""What a context holds on the device: the arrays that its launches read, not the
scratch memory of their preparation (bytes a voxel of source and target of one
size, and a few allocation granules)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _held(make, count=3):
    import torch
    make().close()  # (the library's own first allocations)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    held = [make() for _ in range(count)]
    torch.cuda.synchronize()
    after = torch.cuda.mem_get_info()[0]
    for r in held:
        r.close()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= before - (4 << 20)
    return (before - after) / count


@pytest.mark.parametrize("score, fov, layout_bytes", [("dice", False, 0.0), ("dice", True, 0.0), ("ncc", True, 24.0),
                                                      ("ncc", False, 24.0)])
def test_a_context_holds_no_scratch(score, fov, layout_bytes):
    import torch
    from paper_2504_19930_amd.binding import Registration
    from paper_2504_19930_amd.config import default_params
    side = 256
    src = torch.randint(0, 2 if score == "dice" else 256, (side,) * 3, dtype=torch.uint8, device="cuda")
    mask = torch.ones_like(src) if fov else None
    held = _held(lambda: Registration(src, src, default_params(score, 64, 4, 10.0, 4.0), src_fov=mask))
    # masks: prepared bytes of both, field, bitmaps and blocks 3.5; images: the x-lerps
    # and tiled octets, with a FOV validity, field, target dwords and blocks 3.3
    assert held <= (3.6 + layout_bytes) * side ** 3 + (8 << 20), held / side ** 3
