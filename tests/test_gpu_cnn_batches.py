"""The network's forward and backward at the batch sizes where the forward
takes another split of its work (8 and 16 pairs) or a weight gradient's last
part of K is partly or wholly empty, against the FP64 oracle at the same
bfloat16 decisions (relative L2 error <= 2e-2, the bound of the network's
other parity tests); a step repeated gives the same bits."""

import numpy as np
import pytest

import synth
from oracle import cnn as ocnn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 7, 8, 17])
def test_batches_match_oracle_and_repeat(B):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19930_amd import binding as smc
    net = smc.Cnn(max_batch=B + 1)
    p32 = ocnn.init_params(11)
    net.set_params(p32)
    xs, keep = [], []
    for b in range(B):
        pr = synth.proposal_pair(seed=50 + b)
        keep += [torch.from_numpy(pr[k]).cuda() for k in ("src", "tgt")]
        net.input(b, smc.volume(keep[-2]), smc.volume(keep[-1]), 1.0)
        xs.append(np.stack([ocnn.downsample(pr["src"]), ocnn.downsample(pr["tgt"])]))
    x = ocnn.bf16(np.stack(xs).astype(np.float16).astype(np.float32)).astype(np.float64)
    n_conv = sum(int(np.prod(s)) for s in ocnn.param_shapes()[:8])
    po = p32.astype(np.float32).copy()
    po[:n_conv] = ocnn.bf16(po[:n_conv])
    po = po.astype(np.float64)
    rel = lambda a, b: float(np.linalg.norm(np.ravel(a) - np.ravel(b)) / np.linalg.norm(np.ravel(b)))
    ref, acts = ocnn.forward(po, x, bf16_acts=True)
    out = net.forward(B)
    assert rel(out, ref) <= 2e-2
    assert np.array_equal(out, net.forward(B))
    rng = np.random.default_rng(B)
    target = np.concatenate([rng.normal(0, 0.5, (B, 6)), rng.uniform(0.01, 0.2, (B, 6))], 1)
    loss, g = net.backward(target, grads=True)
    ref_g = ocnn.backward(po, acts, ocnn.nll_grad(ref, target[:, :6], target[:, 6:]))
    offs = np.cumsum([0] + [int(np.prod(s)) for s in ocnn.param_shapes()])
    for q in range(len(offs) - 1):
        assert rel(g[offs[q]:offs[q + 1]], ref_g[offs[q]:offs[q + 1]]) <= 2e-2, q
    loss2, g2 = net.backward(target, grads=True)
    assert loss2 == loss and np.array_equal(g, g2)
    net.close()
