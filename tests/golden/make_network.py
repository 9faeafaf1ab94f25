"""Recorded outputs of the proposal network on an MI355X.

Activations and the gradients of the pre-activations are rounded to bfloat16,
so the network's outputs depend on the order of its FP32 sums: K = (c_in, kz,
ky, kx) in the forward, (c_out, kz, ky, kx) in the data gradient, 32 consecutive
K an instruction.  The values in ``network.json`` were recorded from kernels that
gathered each operand element by element in that order; the outputs and the
loss of any later kernels are the same bits, and of a gradient the sums over
signed elements are kept, whose FP32 sums may be in another order.

    python tests/golden/make_network.py OUT.json
"""

from __future__ import annotations

import hashlib
import json
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "network.json")

import numpy as np  # noqa: E402

# sizes at which the forward's K falls into other ranges, or its work into others
FORWARD = (1, 2, 3, 4, 5, 7, 8, 11, 15, 16, 20, 33)
BACKWARD = (1, 3, 8, 16, 33)
PROJECTIONS = 8


def inputs():
    """Pairs of 64^3 volumes (whole numbers throughout): ellipsoids with noise."""
    rng = np.random.default_rng(77)
    z, y, x = np.meshgrid(*[np.arange(64)] * 3, indexing="ij")
    pairs = []
    for _ in range(max(FORWARD)):
        pair = []
        for _ in range(2):
            c, a = rng.integers(24, 40, 3), rng.integers(9, 25, 3)
            inside = sum((100 * (v - int(m))) ** 2 // int(r) ** 2 for v, m, r in zip((x, y, z), c, a)) <= 10000
            pair.append((200 * inside + rng.integers(0, 48, inside.shape)).astype(np.uint8))
        pairs.append(pair)
    return pairs


def target(B):
    rng = np.random.default_rng(1000 + B)
    t = np.concatenate([rng.integers(-800, 800, (B, 6)) / 1000.0, rng.integers(1, 200, (B, 6)) / 10000.0], axis=1)
    return t.astype(np.float32)


def signs(part, n):
    return 1.0 - 2.0 * np.random.default_rng(500 + part).integers(0, 2, (PROJECTIONS, n))


def parts():
    chans, sizes = (2, 16, 32, 64, 64), []
    for ci, co in zip(chans[:-1], chans[1:]):
        sizes += [co * ci * 27, co]
    return np.cumsum([0] + sizes + [12 * 4096, 12])


def digest(*arrays):
    h = hashlib.sha256()
    for a in arrays:
        h.update(np.ascontiguousarray(a).tobytes())
    return h.hexdigest()


def record(smc, weights):
    import torch
    pairs = inputs()
    net = smc.Cnn(max_batch=max(FORWARD))
    net.set_params(weights)
    keep = []
    for s, pair in enumerate(pairs):
        keep.append([torch.from_numpy(v).cuda() for v in pair])
        net.input(s, smc.volume(keep[-1][0]), smc.volume(keep[-1][1]), 1.0 / 255.0)
    out = dict(inputs=digest(*[v for p in pairs for v in p]), weights=digest(weights), forward={}, loss={}, grads={})
    for B in FORWARD:
        out["forward"][str(B)] = [float(v) for v in net.forward(B).ravel()]
    cut = parts()
    for B in BACKWARD:
        loss, g = net.backward(target(B), grads=True)
        out["loss"][str(B)] = float(loss)
        rows = []
        for q, (lo, hi) in enumerate(zip(cut[:-1], cut[1:])):
            v = g[lo:hi].astype(np.float64)
            rows.append([float(np.linalg.norm(v))] + [float(e) for e in signs(q, hi - lo) @ v])
        out["grads"][str(B)] = rows
    net.close()
    return out


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())
    from paper_2504_19930_amd import binding, learned

    with open(sys.argv[1], "w") as f:
        json.dump(record(binding, learned.load_weights()), f)
