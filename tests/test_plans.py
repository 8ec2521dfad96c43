"""Launch plans, seen through the size queries of the weight gradients (host-only logic: no GPU needed)."""
from paper_1912_05234_amd import binding


def test_only_plain_shapes_ask_for_no_workspace():
    """Zero means that the plain kernel runs.  A matrix-core plan of one workgroup column has no partial sums, yet a call
    without a workspace must not select it."""
    L = binding.lib()
    for shape in ((2, 70, 17, 19, 70, 3, 3), (4, 12, 20, 37, 1, 3, 3)):
        assert L.cnn_conv_bwd_weight_workspace_bytes(*shape) > 0
        assert L.cnn_conv_bwd_weight_bf16_workspace_bytes(*shape) > 0
    for shape in ((6, 26, 16, 22, 1, 3, 3), (8, 23, 20, 22, 1, 4, 4), (1, 1, 28, 28, 6, 5, 5)):
        assert L.cnn_conv_bwd_weight_bf16_workspace_bytes(*shape) > 0
    assert L.cnn_conv_bwd_weight_workspace_bytes(1, 18, 27, 34, 2, 5, 5) == 0
