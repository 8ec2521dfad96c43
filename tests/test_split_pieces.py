"""The estimate of missing products of pieces (split_pieces.py), on results made without one of them."""
import numpy as np
import pytest
import torch

import split_pieces
from paper_1912_05234_amd import inputs


def test_pieces_add_up():
    x = torch.from_numpy(inputs.make_signed((4096,), 3).astype(np.float32))
    assert torch.equal(sum(split_pieces.pieces(x)), x.double())


@pytest.mark.parametrize("lost", [None, 0, 1, 2, 3, 4])
def test_a_missing_product_is_found(lost):
    """Activations of 32 images, rounded to fp32: the product that is left out, and no other."""
    w = {n: torch.from_numpy(v) for n, v in inputs.make_random_biases(inputs.make_weights(), 5).items()}
    x = torch.from_numpy(inputs.make_batch(32, 6)[0].astype(np.float32)).view(32, 1, 28, 28)
    want, without = split_pieces.layer(x, 4.0 * w["k1"].view(6, 1, 5, 5), w["b1"], -split_pieces.LOG2E)
    got = (want if lost is None else without[lost]).float()
    share = split_pieces.missing(got.numpy(), want.numpy(), [a.numpy() for a in without])
    expected = [1.0 if i == lost else 0.0 for i in range(5)]
    np.testing.assert_allclose(share, expected, atol=0.05)


@pytest.mark.parametrize("lost", [None, 0, 1, 2, 3, 4])
def test_a_missing_product_is_found_in_gradients(lost):
    """Both gradients of 520 images, off by an fp32 sum's error (5e-8 of the root mean square)."""
    images, labels = inputs.make_batch(520, 7)
    both = split_pieces.gradients(inputs.make_random_biases(inputs.make_weights(), 8), (2.0 * images - 1.0).astype(np.float32), labels)
    rng = np.random.default_rng(9)
    for want, without in both:
        got = (want if lost is None else without[lost]) + 5e-8 * np.sqrt((want * want).mean()) * rng.standard_normal(want.shape)
        share = split_pieces.missing(got, want, without)
        np.testing.assert_allclose(share, [1.0 if i == lost else 0.0 for i in range(5)], atol=0.15)
