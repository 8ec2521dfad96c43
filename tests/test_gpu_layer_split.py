"""The second convolution's calls on more than 1024 images (one wave per image) against the plain kernels, which test_gpu_ops.py
pins to the oracle: sizes around a whole number of images per wave and workgroup, and operands far from 1; and sums of
one, two and three products against 64 bits, where nothing averages an inexact product away."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1912_05234_amd import binding, inputs
from parity import RTOL_ACT, RTOL_GRAD, assert_close

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).to("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


# The scales are powers of two: the plain kernel's result for operands around 1, scaled, is its result for them.
@pytest.mark.parametrize("B,scale", [(1025, 2.0**-100), (2047, 1.0), (2048, 1.0), (2049, 2.0**100), (4101, 1.0), (18433, 1.0)])
def test_against_the_plain_kernels(B, scale):
    x, k, b, d = (inputs.make_signed(s, 71 + i) for i, s in enumerate([(B, 6, 12, 12), (12, 6, 5, 5), (12,), (B, 12, 8, 8)]))
    xs, ds = dev(x * scale), dev(d * scale)
    x, k, d = dev(x), dev(k), dev(d)
    for bias in (None, b):
        want = host(binding.conv_fwd(x, k, None if bias is None else dev(b), valu=True))
        got = binding.conv_fwd(xs, k, None if bias is None else dev(b * scale))
        assert_close(host(got) / scale, want, RTOL_ACT, "many images conv_fwd")
    assert_close(host(binding.conv_bwd_input(ds, k, 12, 12)) / scale, host(binding.conv_bwd_input(d, k, 12, 12, valu=True)), RTOL_ACT,
                 "many images conv_bwd_input")
    p_k, p_b = binding.conv_bwd_weight(x, d, workspace=False)
    for in_, d_out in ((xs, d), (x, ds)):
        d_k, d_b = binding.conv_bwd_weight(in_, d_out)
        assert_close(host(d_k) / scale, host(p_k), RTOL_GRAD, "many images conv_bwd_weight")
        assert_close(host(d_b) / (scale if d_out is ds else 1.0), host(p_b), RTOL_GRAD, "many images conv_bwd_bias")


def test_weight_gradient_stays_in_its_workspace():
    """Partial sums fit the announced size, and where they do not the plain kernel is taken."""
    B = 2049
    x, d = dev(inputs.make_signed((B, 6, 12, 12), 81)), dev(inputs.make_signed((B, 12, 8, 8), 82))
    p_k, p_b = binding.conv_bwd_weight(x, d, workspace=False)
    L, ptr = binding.lib(), lambda t: ctypes.c_void_p(t.data_ptr())
    need = L.cnn_conv_bwd_weight_workspace_bytes(B, 6, 12, 12, 12, 5, 5)
    for size in (need - 1, need):
        ws = torch.full((need + 4096,), 255, dtype=torch.uint8, device="cuda:0")  # NaN wherever it is read before written
        d_k, d_b = torch.empty_like(p_k), torch.empty_like(p_b)
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert L.cnn_conv_bwd_weight(ptr(x), ptr(d), ptr(d_k), ptr(d_b), B, 6, 12, 12, 12, 5, 5, ptr(ws), ctypes.c_size_t(size), stream) == 0
        assert_close(host(d_k), host(p_k), RTOL_GRAD, "many images conv_bwd_weight")
        assert_close(host(d_b), host(p_b), RTOL_GRAD, "many images conv_bwd_bias")
        used = (ws != 255).nonzero()
        assert used.numel() == 0 or int(used.max()) < size


U = 2.0**-24  # largest relative error of one rounding to fp32


@pytest.mark.parametrize("scale", [1.0, 2.0**-116])
@pytest.mark.parametrize("near_one", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3])
def test_sums_of_few_products(n, near_one, scale):
    """Every result is a sum of n products (at the border of the input gradient fewer), each rounded at most twice (its own
    product, and the sum with what was there before), so off by at most 2 n - 1 roundings of the sum of magnitudes.  Operands
    near 1 have all low bits at work; the small scale is below 2^-109, where a third bfloat16 piece loses bits."""
    rng, B = np.random.default_rng(90 + n), 1300
    sign = lambda s: rng.choice([-1.0, 1.0], s)
    draw = lambda *s: ((1.0 + 0.01 * rng.random(s)) if near_one else (0.5 + 0.5 * rng.random(s))).astype(np.float32) * sign(s).astype(np.float32)
    x, d, k = draw(B, 6, 12, 12), draw(B, 12, 8, 8), draw(12, 6, 5, 5)
    taps, flat, pixels = np.zeros((12, 150), np.float32), np.zeros((6, 300), np.float32), np.zeros((B, 12, 64), np.float32)
    for j in range(12):
        at = rng.permutation(150)[:n]
        taps[j, at] = k.reshape(12, 150)[j, at]
        for image, p in zip(rng.permutation(B)[:n], rng.integers(0, 64, n)):
            pixels[image, j, p] = d.reshape(B, 12, 64)[image, j, p]
    for c in range(6):
        at = rng.permutation(300)[:n]
        flat[c, at] = k.transpose(1, 0, 2, 3).reshape(6, 300)[c, at]
    back, few = np.ascontiguousarray(flat.reshape(6, 12, 5, 5).transpose(1, 0, 2, 3)), pixels.reshape(B, 12, 8, 8)
    taps = taps.reshape(12, 6, 5, 5)

    def fwd64(x, k):
        cols = torch.nn.functional.unfold(torch.from_numpy(x.astype(np.float64)), 5)
        return torch.matmul(torch.from_numpy(k.astype(np.float64)).view(12, 150), cols).view(-1, 12, 8, 8).numpy()

    def in64(d, k):
        t = torch.matmul(torch.from_numpy(k.astype(np.float64)).view(12, 150).t(), torch.from_numpy(d.astype(np.float64)).view(-1, 12, 64))
        return torch.nn.functional.fold(t, (12, 12), 5).numpy()

    def weight64(x, d):
        used = np.flatnonzero(np.abs(d).sum(axis=(1, 2, 3)))
        cols = torch.nn.functional.unfold(torch.from_numpy(x[used].astype(np.float64)), 5)
        return torch.einsum("njp,nip->ji", torch.from_numpy(d[used].astype(np.float64)).view(-1, 12, 64), cols).view(12, 6, 5, 5).numpy()

    xs, ds, fs = (a * np.float32(scale) for a in (x, d, few))  # exact
    for name, got, want, most in [("conv_fwd", binding.conv_fwd(dev(xs), dev(taps)), fwd64(xs, taps), fwd64(abs(xs), abs(taps))),
                                  ("conv_bwd_input", binding.conv_bwd_input(dev(ds), dev(back), 12, 12), in64(ds, back), in64(abs(ds), abs(back))),
                                  ("conv_bwd_weight", binding.conv_bwd_weight(dev(x), dev(fs))[0], weight64(x, fs), weight64(abs(x), abs(fs)))]:
        off = np.abs(host(got) - want)
        worst = (off[most > 0] / most[most > 0]).max() / U
        assert worst <= (2 * n - 1) * 1.01 and not off[most == 0].any(), "%s: %.2f roundings" % (name, worst)
