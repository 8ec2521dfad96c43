"""The second convolution's calls on more than 1024 images (one wave per image, products of bfloat16 pieces) against the plain
kernels, which test_gpu_ops.py pins to the oracle: sizes around a whole number of images per wave and workgroup, and operands
far from 1, where the pieces have to keep a float's range."""
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
        assert_close(host(got) / scale, want, RTOL_ACT, "pieces conv_fwd")
    assert_close(host(binding.conv_bwd_input(ds, k, 12, 12)) / scale, host(binding.conv_bwd_input(d, k, 12, 12, valu=True)), RTOL_ACT,
                 "pieces conv_bwd_input")
    p_k, p_b = binding.conv_bwd_weight(x, d, workspace=False)
    for in_, d_out in ((xs, d), (x, ds)):
        d_k, d_b = binding.conv_bwd_weight(in_, d_out)
        assert_close(host(d_k) / scale, host(p_k), RTOL_GRAD, "pieces conv_bwd_weight")
        assert_close(host(d_b) / (scale if d_out is ds else 1.0), host(p_b), RTOL_GRAD, "pieces conv_bwd_bias")


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
        assert_close(host(d_k), host(p_k), RTOL_GRAD, "pieces conv_bwd_weight")
        assert_close(host(d_b), host(p_b), RTOL_GRAD, "pieces conv_bwd_bias")
        used = (ws != 255).nonzero()
        assert used.numel() == 0 or int(used.max()) < size
