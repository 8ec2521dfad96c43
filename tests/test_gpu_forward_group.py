"""The forward pass with eight waves per image (small batches) on both sides of the line where one wave per image takes
over: the two forms have to agree, and the evaluation with them."""
import numpy as np
import pytest
import torch

from paper_1912_05234_amd import binding, inputs
from parity import RTOL_ACT, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 255, 1536])
def test_forward_and_evaluation(B):
    images, labels = inputs.make_batch(1537, 91)
    net = binding.CNN(inputs.make_random_biases(inputs.make_weights(), 92), max_batch=1537)
    x, lab = torch.from_numpy(images).to("cuda:0"), torch.from_numpy(labels).to("cuda:0")
    one_wave = net.forward_activations(x)
    group = net.forward_activations(x[:B])
    y = net.forward(x[:B])
    n_ok, loss = net.evaluate(x[:B], lab[:B])
    torch.cuda.synchronize()
    for name in ("c1", "s1", "c2", "s2", "y"):
        assert_close(group[name].cpu().numpy(), one_wave[name][:B].cpu().numpy().astype(np.float64), RTOL_ACT, name)
    assert torch.equal(y, group["y"])
    y64 = y.cpu().numpy().astype(np.float64)
    assert int(n_ok[0]) == int((y64.argmax(axis=1) == labels[:B]).sum())
    want = 0.5 * float(((y64 - np.eye(10)[labels[:B]]) ** 2).sum())
    assert abs(float(loss[0]) - want) <= 1e-5 * want
