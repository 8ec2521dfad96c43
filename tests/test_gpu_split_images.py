"""The network's own convolution layers on few images, where several waves share one: on both sides of the lines where the
split changes, against the plain kernels, which test_gpu_ops.py pins to the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1912_05234_amd import binding, inputs
from parity import RTOL_ACT, RTOL_GRAD, assert_close

pytestmark = pytest.mark.gpu

LAYERS = {"c1": (1, 28, 6), "c2": (6, 12, 12)}  # input maps, extent, output maps; 5 x 5 taps


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("B", [1, 2, 3, 255, 256, 257, 1023, 1024, 1025])
@pytest.mark.parametrize("layer", sorted(LAYERS))
def test_split_layers(layer, B):
    cin, n, cout = LAYERS[layer]
    x, k, b = dev(inputs.make_signed((B, cin, n, n), 61)), dev(inputs.make_signed((cout, cin, 5, 5), 62)), dev(inputs.make_signed((cout,), 63))
    d = dev(inputs.make_signed((B, cout, n - 4, n - 4), 64))
    assert_close(host(binding.conv_fwd(x, k, b)), host(binding.conv_fwd(x, k, b, valu=True)), RTOL_ACT, "split conv_fwd")
    assert_close(host(binding.conv_bwd_input(d, k, n, n)), host(binding.conv_bwd_input(d, k, n, n, valu=True)), RTOL_ACT, "split conv_bwd_input")
    d_k, d_b = binding.conv_bwd_weight(x, d)
    p_k, p_b = binding.conv_bwd_weight(x, d, workspace=False)
    assert_close(host(d_k), host(p_k), RTOL_GRAD, "split conv_bwd_weight")
    assert_close(host(d_b), host(p_b), RTOL_GRAD, "split conv_bwd_bias")


@pytest.mark.parametrize("B", [1, 9, 256, 1024])
@pytest.mark.parametrize("layer", sorted(LAYERS))
def test_weight_gradient_in_a_smaller_workspace(layer, B):
    """Partial sums of one workgroup per eight images, as many as without the split, are enough; a byte less is not."""
    cin, n, cout = LAYERS[layer]
    x, d = dev(inputs.make_signed((B, cin, n, n), 65)), dev(inputs.make_signed((B, cout, n - 4, n - 4), 66))
    p_k, p_b = binding.conv_bwd_weight(x, d, workspace=False)
    row = 4 * (16 + 256 * (2 if layer == "c1" else 10))
    least = row * -(-B // 8)
    L, ptr = binding.lib(), lambda t: ctypes.c_void_p(t.data_ptr())
    assert L.cnn_conv_bwd_weight_workspace_bytes(B, cin, n, n, cout, 5, 5) >= least
    for size in (least - 1, least, least + row - 1):
        ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device="cuda:0")  # NaN wherever it is read before written
        d_k, d_b = torch.empty_like(p_k), torch.empty_like(p_b)
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert L.cnn_conv_bwd_weight(ptr(x), ptr(d), ptr(d_k), ptr(d_b), B, cin, n, n, cout, 5, 5, ptr(ws), ctypes.c_size_t(size), stream) == 0
        assert_close(host(d_k), host(p_k), RTOL_GRAD, "split conv_bwd_weight")
        assert_close(host(d_b), host(p_b), RTOL_GRAD, "split conv_bwd_bias")
        used = (ws != 255).nonzero()
        assert size >= least or used.numel() == 0
        assert used.numel() == 0 or int(used.max()) < size
