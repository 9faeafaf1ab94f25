"""The proposal network's outputs and loss are the recorded bits at every size
where the forward splits its sums or its work differently, and its gradients the
recorded ones up to the order of the weight gradients' FP32 sums: chains of up to
2048 additions, whose roundings add up to some 2^-24 sqrt(2048) = 2.7e-6 of a
part's norm (4e-6 allowed).  Another order of the sums in front of a
rounding to bfloat16 moves them by 1e-5 and more."""

import importlib.util
import json
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
_spec = importlib.util.spec_from_file_location("make_network", os.path.join(HERE, "golden", "make_network.py"))
golden = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(golden)


@pytest.fixture(scope="module")
def recorded():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_19930_amd import binding, learned
    now = golden.record(binding, learned.load_weights())
    with open(golden.OUT) as f:
        then = json.load(f)
    assert now["inputs"] == then["inputs"] and now["weights"] == then["weights"]
    return now, then


@pytest.mark.parametrize("B", golden.FORWARD)
def test_outputs_are_the_recorded_bits(recorded, B):
    now, then = recorded
    assert now["forward"][str(B)] == then["forward"][str(B)]


@pytest.mark.parametrize("B", golden.BACKWARD)
def test_loss_and_gradients_are_the_recorded_ones(recorded, B):
    now, then = recorded
    assert now["loss"][str(B)] == then["loss"][str(B)]
    for q, (a, b) in enumerate(zip(now["grads"][str(B)], then["grads"][str(B)])):
        assert np.all(np.abs(np.array(a) - np.array(b)) <= 4e-6 * b[0]), (q, a, b)
