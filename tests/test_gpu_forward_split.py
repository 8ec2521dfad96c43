"""The forward pass of more than 1024 images and the gradient of more than 512 (one wave per image, convolutions as products
of bfloat16 pieces) against the fp32 matrix instructions that smaller calls run on: sizes around a whole number of images per wave and workgroup, and
operands far from 1, where the pieces have to keep a float's range; and against 64 bits, where a product of pieces that is left
out shows."""
import numpy as np
import pytest
import torch

import split_pieces
from paper_1912_05234_amd import binding, inputs
from parity import RTOL_ACT, RTOL_GRAD, assert_close

pytestmark = pytest.mark.gpu


# Pixels times `gain`, the factor on k1, stay around 1, so that C1 depends on both; `upper` is the factor on k2 and fc.
@pytest.mark.parametrize("B,pixel,gain,upper", [(1025, 1.0, 1.0, 1.0), (2048, 1e-3, 1e3, 4.0), (2049, 1.0, 4.0, 4.0),
                                                (4101, 3e4, 1e-4, 0.25), (1031, 1e-30, 1e30, 1.0), (1033, 1e30, 1e-30, 4.0)])
def test_against_the_fp32_instructions(B, pixel, gain, upper):
    images, labels = inputs.make_batch(B, 17)
    images = images * np.float32(pixel)
    w = inputs.make_random_biases(inputs.make_weights(), 18)
    for name in ("k1", "k2", "fc"):
        w[name] = (w[name] * np.float32(gain if name == "k1" else upper)).astype(np.float32)
    net = binding.CNN(w, max_batch=B)
    x = torch.from_numpy(images).to("cuda:0")
    got = net.forward_activations(x)
    parts = [net.forward_activations(x[i:i + 1000]) for i in range(0, B, 1000)]
    for name in ("c1", "s1", "c2", "s2", "y"):
        want = torch.cat([p[name] for p in parts]).cpu().numpy().astype(np.float64)
        assert_close(got[name].cpu().numpy(), want, RTOL_ACT, "split " + name)
    y = net.forward(x)
    n_ok, loss = net.evaluate(x, torch.from_numpy(labels).to("cuda:0"))
    assert torch.equal(y, got["y"])
    y64 = y.cpu().numpy().astype(np.float64)
    assert int(n_ok[0]) == int((y64.argmax(axis=1) == labels).sum())
    want = 0.5 * float(((y64 - np.eye(10)[labels]) ** 2).sum())
    assert abs(float(loss[0]) - want) <= 1e-5 * want


def test_updated_weights_reach_the_pieces():
    """After a training step the pieces are those of the new weights."""
    images, labels = inputs.make_batch(1100, 19)
    net = binding.CNN(inputs.make_weights(), max_batch=1100)
    x, lab = torch.from_numpy(images).to("cuda:0"), torch.from_numpy(labels).to("cuda:0")
    for n in (100, 1100):
        net.train_batch(x[:n].contiguous(), lab[:n].contiguous(), 2.0)
    fresh = binding.CNN(net.get_weights(), max_batch=1100)
    assert torch.equal(net.forward(x), fresh.forward(x))


# (3585 images: fourteen and fifteen to a workgroup, dealt to its waves in three rounds)
@pytest.mark.parametrize("B,pixel,gain", [(513, 1.0, 1.0), (641, 1.0, 1.0), (1025, 1e-3, 1e3), (2049, 1.0, 4.0), (3585, 1.0, 1.0),
                                          (1100, 1e30, 1e-30), (700, 1e-30, 1e30)])
def test_gradient_against_the_fp32_instructions(B, pixel, gain):
    images, labels = inputs.make_batch(B, 27)
    w = inputs.make_random_biases(inputs.make_weights(), 28)
    w["k1"] = (w["k1"] * np.float32(gain)).astype(np.float32)
    net = binding.CNN(w, max_batch=B)
    x, lab = torch.from_numpy(images * np.float32(pixel)).to("cuda:0"), torch.from_numpy(labels).to("cuda:0")
    grad, loss = (t.cpu().numpy().astype(np.float64) for t in net.gradient(x, lab))
    want, want_loss = np.zeros_like(grad), 0.0
    for i in range(0, B, 500):
        g, n = net.gradient(x[i:i + 500].contiguous(), lab[i:i + 500].contiguous())
        want += g.cpu().numpy().astype(np.float64)
        want_loss += float(n.cpu().numpy().sum())
    at = 0
    for name, shape in inputs.PARAM_SHAPES:
        n = int(np.prod(shape))
        assert_close(grad[at:at + n], want[at:at + n], RTOL_GRAD, "split grad " + name)
        at += n
    assert abs(loss.sum() - want_loss) <= 1e-5 * want_loss


# A product that is left out has a share of 1.  The results' own rounding, of another pattern than any product, gives shares of up
# to 0.05 in the gradients (150 and 1800 weights) and 0.005 in the activations.
SHARE = 0.25


def test_activations_have_every_product():
    B = 1025
    images, w = inputs.make_batch(B, 37)[0], inputs.make_random_biases(inputs.make_weights(), 38)
    for name in ("k1", "k2"):
        w[name] = (4.0 * w[name]).astype(np.float32)
    net = binding.CNN(w, max_batch=B)
    got = {n: t.cpu() for n, t in net.forward_activations(torch.from_numpy(images).to("cuda:0")).items()}
    t = {n: torch.from_numpy(v) for n, v in w.items()}
    for name, x, k, b, pooled in (("c1", torch.from_numpy(images).view(B, 1, 28, 28), t["k1"].view(6, 1, 5, 5), t["b1"], 1.0),
                                  ("c2", got["s1"].view(B, 6, 12, 12), t["k2"].view(12, 6, 5, 5), t["b2"], 0.25)):
        want, without = split_pieces.layer(x, k, b, -split_pieces.LOG2E, pooled)
        share = split_pieces.missing(got[name].view(want.shape).numpy(), want.numpy(), [a.numpy() for a in without])
        print(name, share)
        assert np.abs(share).max() <= SHARE, (name, share)


@pytest.mark.parametrize("B", [600, 1100])
def test_gradients_have_every_product(B):
    images, labels = inputs.make_batch(B, 39)
    images, w = (2.0 * images - 1.0).astype(np.float32), inputs.make_random_biases(inputs.make_weights(), 40)
    net = binding.CNN(w, max_batch=B)
    grad = net.gradient(torch.from_numpy(images).to("cuda:0"), torch.from_numpy(labels).to("cuda:0"))[0].cpu().numpy()
    (k2, without_k2), (k1, without_k1) = split_pieces.gradients(w, images, labels)
    for name, got, want, without in (("k1", grad[:150], k1, without_k1), ("k2", grad[156:1956], k2, without_k2)):
        share = split_pieces.missing(got, want, without)
        print(name, share)
        assert np.abs(share).max() <= SHARE, (name, share)


def sigmoid(z):
    return 1.0 / (1.0 + np.exp(-z))


@pytest.mark.parametrize("low", [1.0 + 2.0**-7 - 2.0**-14, 1.0 + 2.0**-8 - 2.0**-17])
def test_left_out_products_stay_below_a_rounding(low):
    """Pixels and weights just below the next bfloat16, or just below the middle of two, where what the cut leaves out is largest
    and of one sign in every product.  Each operand's second and third pieces are at most 2^-8 and 2^-17 of its power of
    two, so the two products left out are at most 2^-24 of the product's; the constant log2(e), with which the weights are
    multiplied before the cut, is off by 0.22 x 2^-24 as a float; the other roundings have no common sign.
    Measured as the factor by which the sums before the sigmoid are off, over all of C1."""
    rng, B = np.random.default_rng(7), 1025
    w = {"k1": np.zeros((6, 5, 5), np.float32)}
    w["k1"][:] = 2.0**-4 * np.where(np.arange(6) % 2, 1.0, -1.0)[:, None, None] * (low + 2.0**-16 * rng.random((6, 5, 5))) / np.log2(np.e)
    images = (low + 2.0**-16 * rng.random((B, 28, 28))).astype(np.float32)
    images[:, :, ::2] = 0.0  # sums around 1, where the sigmoid is steep
    net = binding.CNN(w, max_batch=B)
    got = net.forward_activations(torch.from_numpy(images).to("cuda:0"))["c1"].cpu().numpy().astype(np.float64)
    k = torch.from_numpy(w["k1"].astype(np.float64)).view(6, 25)
    z = torch.matmul(k, torch.nn.functional.unfold(torch.from_numpy(images.astype(np.float64)).view(B, 1, 28, 28), 5)).numpy().reshape(got.shape)
    steep = z * sigmoid(z) * sigmoid(-z)
    off = ((got - sigmoid(z)) * steep).sum() / (steep * steep).sum()
    assert abs(off) <= 1.5 * 2.0**-24, "sums off by %.2f x 2^-24" % (off * 2.0**24)
