"""Preparation of a pair at the edges of its kernels: volumes at odd addresses
(wide loads), sizes with remainders in 16-byte loads, 64-voxel ballots and 4^3
blocks, and sources that hold the values which mark octets outside the FOV.

Sums over every voxel are whole numbers, so equal to the oracle's; one
iteration's log-weights come from whole counts by one FP64 formula (1e-12
relative, 1e-10 for correlations, which divide differences of large sums)."""

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


def _at(a, offset):
    """A contiguous device tensor of a's values that starts `offset` bytes past an aligned address."""
    import torch
    flat = torch.empty(a.size + offset, dtype=torch.uint8, device="cuda")
    out = flat[offset:].view(a.shape)
    out.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    return out


@pytest.mark.parametrize("score", ["dice", "ncc"])
@pytest.mark.parametrize("offsets", [(0, 0), (1, 1), (0, 3), (7, 0)])  # volumes, FOVs
@pytest.mark.parametrize("shape", [(1, 1, 2), (3, 5, 7), (17, 16, 64), (9, 13, 65), (20, 31, 66)])
def test_statistics_at_odd_addresses_and_sizes(smc, orc, score, offsets, shape):
    rng = np.random.default_rng(4)
    draw = lambda: rng.integers(0, 2 if score == "dice" else 256, shape).astype(np.uint8)
    src, tgt = draw(), draw()
    sfov, tfov = (rng.random(shape) < 0.97).astype(np.uint8), (rng.random(shape) < 0.8).astype(np.uint8)
    tfov.flat[0] = 200  # any value but 0 is inside
    prm = config.default_params(score, 40, 1, 10.0, 1.0, seed=2)
    v, f = offsets
    r = smc.Registration(_at(src, v), _at(tgt, v), prm, src_fov=_at(sfov, f), tgt_fov=_at(tfov, f))
    r.run()
    o = orc.smc_run(orc.Volume(src, fov=sfov), orc.Volume(tgt, fov=tfov), prm)
    tol = 1e-12 if score == "dice" else 1e-10
    assert np.allclose(r.particles()["logw"], o["logw"], rtol=tol, atol=tol)
    r.close()


def _splitmix64(x):
    m = (1 << 64) - 1
    x = (x + 0x9E3779B97F4A7C15) & m
    x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & m
    x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & m
    return x ^ (x >> 31)


@pytest.mark.parametrize("taken", [1, 3, 64])  # of the 64 values tried: one left over or none
def test_sources_that_hold_the_marking_values(smc, orc, taken):
    rng = np.random.default_rng(5)
    src = rng.integers(0, 256, (16, 18, 20)).astype(np.uint8)
    for q in range(taken):  # the 2^3 cell at an even corner holds value q, x fastest
        z, y, x = 2 * (q // 32), 2 * ((q // 8) % 4), 2 * (q % 8)
        cell = np.frombuffer(np.uint64(_splitmix64(q + 1)).tobytes(), np.uint8).reshape(2, 2, 2)
        src[z:z + 2, y:y + 2, x:x + 2] = cell
    fov = np.ones(src.shape, np.uint8)
    fov[12:, :, :] = 0
    fov[:, :, 18:] = 0
    tgt = rng.integers(0, 256, (15, 16, 17)).astype(np.uint8)
    states = np.concatenate([np.deg2rad(rng.uniform(-20, 20, (30, 3))), rng.uniform(-3, 3, (30, 3))], 1)
    states[0] = 0.0  # samples the cells themselves
    prm = config.default_params("ncc", 30, 1, 20.0, 3.0, seed=1)
    r = smc.Registration(_at(src, 0), _at(tgt, 0), prm, src_fov=_at(fov, 0))
    s, t = orc.Volume(src, fov=fov), orc.Volume(tgt)
    want = np.array([orc.image_moments(s, t, orc.recipe_words(p, s, t, nn=False), True) for p in states], dtype=np.int64)
    for layout in ("lerp", "octtile", "oct", "quadxy", "pairx"):
        r.tune(layout)
        assert np.array_equal(r.evaluate(states), want), layout
    r.run()
    o = orc.smc_run(s, t, prm)
    assert np.allclose(r.particles()["logw"], o["logw"], rtol=1e-10, atol=1e-10)
    r.close()
