"""The image-tiled convolution kernels where their cutting can go wrong: ragged bands, strips of very wide images,
channel chunks, several row blocks, packed columns that do not divide a row, one workgroup column, images beyond
64 KB.  Forward and input gradient against the plain kernels, which test_gpu_ops.py pins to the oracle; the weight gradient,
of which small calls run the plain kernel themselves, against a double-precision sum on the host."""
import numpy as np
import pytest
import torch

import oracle
from paper_1912_05234_amd import binding, inputs
from parity import RTOL_ACT, assert_close

pytestmark = pytest.mark.gpu

# (B, Cin, H, W, Cout, KH, KW)
CASES = [(2, 3, 9, 700, 5, 3, 3), (1, 1, 3, 2500, 1, 3, 3),            # strips (weight gradient: the plain kernel)
         (70, 3, 9, 700, 5, 3, 3), (66, 1, 4, 1000, 3, 3, 3),           # wide rows, bands of one of them
         (2, 70, 17, 19, 70, 3, 3), (1, 300, 9, 9, 5, 3, 3),            # chunks, several row blocks and tap groups (the second's
                                                                        # weight gradient: the plain kernel)
         (33, 3, 32, 32, 16, 5, 5), (70, 16, 28, 28, 32, 3, 3),         # bands with a ragged last one, two row tiles
         (40, 2, 11, 7, 3, 2, 3), (5, 1, 13, 27, 2, 7, 7), (9, 2, 14, 7, 1, 5, 5),  # packed, ragged rows
         (301, 4, 30, 13, 4, 3, 3), (1100, 5, 6, 9, 7, 1, 1),           # several images per unit, a ragged last group
         (1, 18, 27, 34, 2, 5, 5), (6, 26, 16, 22, 1, 3, 3),            # few images, few maps (weight gradient: the plain kernel)
         (4, 16, 13, 40, 1, 3, 3), (5, 30, 12, 14, 64, 3, 3),           # weight gradients of one workgroup column (no second kernel;
                                                                        # and 2 images 70 -> 70 above)
         (70, 300, 9, 9, 5, 3, 3),                                      # many tap groups
         (3, 12, 70, 60, 9, 4, 6)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def weight_gradient(x, d, KH, KW):
    """`backweights` and `backbias` summed over the batch, in double precision on the host."""
    x, d = x.astype(np.float64), d.astype(np.float64)
    Ho, Wo = d.shape[2:]
    k = np.empty((d.shape[1], x.shape[1], KH, KW))
    for u in range(KH):
        for v in range(KW):
            k[:, :, u, v] = np.tensordot(d, x[:, :, u:u + Ho, v:v + Wo], axes=((0, 2, 3), (0, 2, 3)))
    return k, d.sum(axis=(0, 2, 3))


@pytest.mark.parametrize("case", CASES)
def test_tiled_convolutions(case):
    B, Cin, H, W, Cout, KH, KW = case
    x, d = inputs.make_signed((B, Cin, H, W), 71), inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 74)
    p_k, p_b = weight_gradient(x, d, KH, KW)
    x, d = dev(x), dev(d)
    k = dev(inputs.make_signed((Cout, Cin, KH, KW), 72))
    b = dev(inputs.make_signed((Cout,), 73))
    assert_close(host(binding.conv_fwd(x, k, b)), host(binding.conv_fwd(x, k, b, valu=True)).astype(np.float64), RTOL_ACT, "tiled conv_fwd")
    assert_close(host(binding.conv_bwd_input(d, k, H, W)), host(binding.conv_bwd_input(d, k, H, W, valu=True)).astype(np.float64),
                 RTOL_ACT, "tiled conv_bwd_input")
    for workspace in (True, False):
        d_k, d_b = binding.conv_bwd_weight(x, d, workspace=workspace)
        assert_close(host(d_k), p_k, RTOL_ACT, "tiled conv_bwd_weight")
        assert_close(host(d_b), p_b, RTOL_ACT, "tiled conv_bwd_bias")
    d_k, _ = binding.conv_bwd_weight(x, d)
    again, none = binding.conv_bwd_weight(x, d, want_bias=False)
    assert none is None and torch.equal(again, d_k)


# Without a workspace the plain kernel runs, whatever the plan: an infinity reaches the weights that meet it and no others.
# (One workgroup column each; the matrix-core kernel multiplies the rows' ends of the first by zero for other taps, and
# cells of the others for padding steps.)
@pytest.mark.parametrize("case,pixel", [((4, 16, 13, 40, 1, 3, 3), (3, 11, 7, 0)), ((2, 70, 17, 19, 70, 3, 3), (1, 5, 0, 0)),
                                        ((6, 26, 16, 22, 1, 3, 3), (0, 25, 0, 0))])
@pytest.mark.parametrize("bf16", [False, True])
def test_weight_gradient_without_workspace_keeps_infinities_local(case, pixel, bf16):
    B, Cin, H, W, Cout, KH, KW = case
    Ho, Wo = H - KH + 1, W - KW + 1
    x, d = oracle.round_bf16(inputs.make_signed((B, Cin, H, W), 95)), oracle.round_bf16(inputs.make_signed((B, Cout, Ho, Wo), 96))
    x[pixel] = np.inf
    ref, ref_b = weight_gradient(x, d, KH, KW)
    assert not np.isnan(ref).any()  # one infinity and no zeros: every sum has a value
    d_k, d_b = binding.conv_bwd_weight(dev(x), dev(d), workspace=False, bf16=bf16)
    d_k, hit = host(d_k), np.isinf(ref)
    assert 0 < hit.sum() < hit.size and np.array_equal(d_k[hit], ref[hit].astype(np.float32))
    assert_close(d_k[~hit], ref[~hit], RTOL_ACT, "conv_bwd_weight beside an infinity")
    assert_close(host(d_b), ref_b, RTOL_ACT, "conv_bwd_bias beside an infinity")


# Weight gradients with five tap tiles per workgroup, one and two row tiles; the blocks of sixteen pixels that a wave
# takes are one, two (a whole trip), three and more, and not the same for all waves.  And layers of as many taps
# whose workgroups would take a unit each, with other tiles.
@pytest.mark.parametrize("case", [(1386, 8, 27, 7, 3, 7, 7), (971, 4, 8, 27, 10, 7, 7), (316, 20, 19, 30, 4, 2, 2), (600, 20, 37, 7, 3, 7, 7),
                                  (1855, 17, 10, 12, 4, 3, 3), (120, 17, 36, 34, 19, 2, 2), (315, 8, 21, 24, 19, 3, 3), (166, 4, 39, 16, 18, 7, 7),
                                  (39, 16, 35, 39, 17, 5, 5),
                                  (695, 19, 9, 13, 1, 2, 2), (862, 8, 11, 9, 6, 3, 3), (1010, 5, 17, 9, 3, 4, 4), (858, 12, 7, 8, 2, 7, 7),
                                  (731, 17, 7, 16, 19, 2, 2), (169, 17, 18, 24, 20, 2, 2), (307, 17, 23, 13, 15, 5, 5), (427, 17, 11, 15, 12, 5, 5),
                                  (709, 16, 11, 15, 34, 3, 3), (870, 9, 11, 23, 7, 4, 4)])
def test_weight_gradients_of_five_tap_tiles(case):
    B, Cin, H, W, Cout, KH, KW = case
    x, d = inputs.make_signed((B, Cin, H, W), 107), inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 108)
    p_k, p_b = weight_gradient(x, d, KH, KW)
    d_k, d_b = binding.conv_bwd_weight(dev(x), dev(d))
    assert_close(host(d_k), p_k, RTOL_ACT, "conv_bwd_weight of five tap tiles")
    assert_close(host(d_b), p_b, RTOL_ACT, "conv_bwd_bias of five tap tiles")


# Weight gradients whose columns are not packed: planes of d_out in whole fours (16 bytes per lane) or not, several images per
# unit with a ragged last group, bands with a ragged last one, row blocks of one and of many maps, one map of many pixels.
@pytest.mark.parametrize("case", [(301, 3, 6, 6, 12, 3, 3), (70, 3, 30, 30, 20, 3, 3), (50, 2, 9, 8, 17, 2, 3), (65, 2, 9, 9, 16, 3, 3), (7, 4, 40, 40, 9, 5, 5),
                                  (90, 1, 28, 30, 33, 3, 3), (1001, 4, 14, 14, 16, 1, 1), (130, 5, 11, 13, 40, 3, 2), (257, 2, 5, 5, 9, 4, 4),
                                  (66, 3, 20, 300, 12, 1, 3), (5, 30, 12, 14, 64, 3, 3), (200, 1, 28, 28, 1, 1, 1), (80, 3, 41, 21, 1, 1, 1)])
@pytest.mark.parametrize("bf16", [False, True])
def test_unpacked_weight_gradients(case, bf16):
    B, Cin, H, W, Cout, KH, KW = case
    x, d = inputs.make_signed((B, Cin, H, W), 105), inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 106)
    p_k, p_b = weight_gradient(oracle.round_bf16(x) if bf16 else x, oracle.round_bf16(d) if bf16 else d, KH, KW)
    d_k, d_b = binding.conv_bwd_weight(dev(x), dev(d), bf16=bf16)
    assert_close(host(d_k), p_k, RTOL_ACT, "unpacked conv_bwd_weight")
    assert_close(host(d_b), p_b, RTOL_ACT, "unpacked conv_bwd_bias")


# Second kernels of the weight gradients: columns of sixteen, of which a trip takes 512 rows (there are 512 of them, or 768 with rounded
# operands, and 700), and of 64, of which it takes 128 (128, and 153).
@pytest.mark.parametrize("case", [(1000, 3, 32, 32, 16, 5, 5), (700, 2, 30, 30, 5, 3, 3), (90, 16, 28, 28, 64, 3, 3), (200, 32, 20, 20, 32, 3, 3)])
@pytest.mark.parametrize("bf16", [False, True])
def test_second_kernels(case, bf16):
    B, Cin, H, W, Cout, KH, KW = case
    x, d = inputs.make_signed((B, Cin, H, W), 112), inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 113)
    p_k, p_b = weight_gradient(oracle.round_bf16(x) if bf16 else x, oracle.round_bf16(d) if bf16 else d, KH, KW)
    d_k, d_b = binding.conv_bwd_weight(dev(x), dev(d), bf16=bf16)
    assert_close(host(d_k), p_k, RTOL_ACT, "conv_bwd_weight of many rows")
    assert_close(host(d_b), p_b, RTOL_ACT, "conv_bwd_bias of many rows")


# Packed columns whose taps lie in runs of two or four: with and without a border, ragged rows, bands and channel chunks,
# whole images per unit, and (the last two) rows of odd length, which have no runs without a border.
@pytest.mark.parametrize("case", [(33, 3, 28, 32, 3, 5, 5), (500, 3, 32, 32, 15, 5, 5), (130, 2, 20, 11, 25, 5, 5), (18, 5, 33, 33, 2, 3, 3),
                                  (1100, 4, 17, 30, 2, 3, 3), (700, 2, 22, 18, 10, 7, 7), (723, 3, 21, 16, 1, 5, 5), (10, 1, 30, 36, 2, 3, 3),
                                  (95, 3, 10, 40, 14, 5, 5), (60, 2, 13, 15, 3, 3, 5), (60, 5, 9, 35, 3, 5, 5)])
def test_runs_of_taps(case):
    B, Cin, H, W, Cout, KH, KW = case
    x, k, b = inputs.make_signed((B, Cin, H, W), 91), inputs.make_signed((Cout, Cin, KH, KW), 92), inputs.make_signed((Cout,), 93)
    d = inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 94)
    x, k, b, d = dev(x), dev(k), dev(b), dev(d)
    assert_close(host(binding.conv_fwd(x, k, b)), host(binding.conv_fwd(x, k, b, valu=True)).astype(np.float64), RTOL_ACT, "tiled conv_fwd")
    assert_close(host(binding.conv_bwd_input(d, k, H, W)), host(binding.conv_bwd_input(d, k, H, W, valu=True)).astype(np.float64),
                 RTOL_ACT, "tiled conv_bwd_input")


# One tap, columns packed: rows of whole and of ragged columns, several images or bands per unit, more than one chunk of
# channels, one row of pixels, and maps that fill a row tile by themselves.
@pytest.mark.parametrize("case", [(300, 2, 24, 24, 2), (78, 16, 27, 19, 2), (50, 32, 33, 10, 3), (1, 1, 5, 17, 1), (40, 1, 39, 37, 5), (90, 8, 21, 23, 4),
                                  (200, 3, 1, 33, 7), (25, 40, 36, 36, 2), (33, 4, 14, 14, 16)])
@pytest.mark.parametrize("bf16", [False, True])
def test_packed_columns_of_one_tap(case, bf16):
    B, Cin, H, W, Cout = case
    x, k = oracle.round_bf16(inputs.make_signed((B, Cin, H, W), 97)), oracle.round_bf16(inputs.make_signed((Cout, Cin, 1, 1), 98))
    d, b = oracle.round_bf16(inputs.make_signed((B, Cout, H, W), 99)), inputs.make_signed((Cout,), 100)
    x64, k64, d64 = x.astype(np.float64), k[:, :, 0, 0].astype(np.float64), d.astype(np.float64)
    out = np.tensordot(k64, x64, axes=(1, 1)).transpose(1, 0, 2, 3) + b[:, None, None]
    d_in = np.tensordot(k64, d64, axes=(0, 1)).transpose(1, 0, 2, 3)
    assert_close(host(binding.conv_fwd(dev(x), dev(k), dev(b), bf16=bf16)), out, RTOL_ACT, "tiled conv_fwd of one tap")
    assert_close(host(binding.conv_bwd_input(dev(d), dev(k), H, W, bf16=bf16)), d_in, RTOL_ACT, "tiled conv_bwd_input of one tap")


# Whole images of 257 to 384 columns (six column tiles per wave): unpacked, packed with ragged rows, with runs of taps, three
# row blocks, one tap.
@pytest.mark.parametrize("case", [(600, 2, 20, 20, 16, 3), (700, 12, 19, 33, 7, 1), (520, 2, 32, 42, 4, 3), (520, 1, 34, 44, 3, 5), (513, 9, 21, 21, 33, 4),
                                  (800, 4, 30, 46, 2, 1)])
@pytest.mark.parametrize("bf16", [False, True])
def test_six_column_tiles(case, bf16):
    B, Cin, H, W, Cout, K = case
    x, k = oracle.round_bf16(inputs.make_signed((B, Cin, H, W), 107)), oracle.round_bf16(inputs.make_signed((Cout, Cin, K, K), 108))
    x, k, b = dev(x), dev(k), dev(inputs.make_signed((Cout,), 109))
    assert_close(host(binding.conv_fwd(x, k, b, bf16=bf16)), host(binding.conv_fwd(x, k, b, valu=True)).astype(np.float64), RTOL_ACT,
                 "tiled conv_fwd of six column tiles")


# Kernels of many channels or taps: weights that fit in LDS all at once, or only those of a chunk of channels, the last with fewer.
@pytest.mark.parametrize("case", [(3, 100, 13, 14, 6, 7, 7), (4, 31, 40, 40, 31, 7, 7), (3, 60, 20, 20, 2, 5, 5), (2, 6, 13, 14, 100, 7, 7), (40, 3, 32, 32, 15, 5, 5),
                                  (5, 200, 24, 24, 2, 5, 5)])
@pytest.mark.parametrize("bf16", [False, True])
def test_weight_tables(case, bf16):
    B, Cin, H, W, Cout, KH, KW = case
    x, k = oracle.round_bf16(inputs.make_signed((B, Cin, H, W), 85)), oracle.round_bf16(inputs.make_signed((Cout, Cin, KH, KW), 86))
    d, b = oracle.round_bf16(inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 87)), inputs.make_signed((Cout,), 88)
    x, k, d, b = dev(x), dev(k), dev(d), dev(b)
    assert_close(host(binding.conv_fwd(x, k, b, bf16=bf16)), host(binding.conv_fwd(x, k, b, valu=True)).astype(np.float64), RTOL_ACT, "tiled conv_fwd")
    assert_close(host(binding.conv_bwd_input(d, k, H, W, bf16=bf16)), host(binding.conv_bwd_input(d, k, H, W, valu=True)).astype(np.float64),
                 RTOL_ACT, "tiled conv_bwd_input")


# Reduced-precision calls that run an fp32 kernel with rounded operands (few channels, small calls, the network's first
# layer in its three splits), on operands that rounding changes.
@pytest.mark.parametrize("case", [(1, 1, 28, 28, 6, 5, 5), (700, 1, 28, 28, 6, 5, 5), (1500, 1, 28, 28, 6, 5, 5), (680, 2, 29, 22, 2, 3, 3), (100, 1, 40, 40, 1, 7, 7),
                                  (3, 6, 6, 18, 5, 1, 1), (10, 1, 30, 36, 2, 3, 3), (600, 8, 14, 15, 8, 1, 1), (2, 40, 9, 11, 3, 3, 3), (5, 2, 4, 300, 2, 3, 5)])
def test_rounded_operands(case):
    B, Cin, H, W, Cout, KH, KW = case
    x, k, b = inputs.make_signed((B, Cin, H, W), 101), inputs.make_signed((Cout, Cin, KH, KW), 102), dev(inputs.make_signed((Cout,), 103))
    d = inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 104)
    xr, kr, dr = dev(oracle.round_bf16(x)), dev(oracle.round_bf16(k)), dev(oracle.round_bf16(d))
    out, want = host(binding.conv_fwd(dev(x), dev(k), b, bf16=True)), host(binding.conv_fwd(xr, kr, b, valu=True)).astype(np.float64)
    assert_close(out, want, RTOL_ACT, "rounded conv_fwd")
    assert np.abs(host(binding.conv_fwd(dev(x), dev(k), b)) - want).max() > 20 * np.abs(out - want).max()
    d_in, want = host(binding.conv_bwd_input(dev(d), dev(k), H, W, bf16=True)), host(binding.conv_bwd_input(dr, kr, H, W, valu=True)).astype(np.float64)
    assert_close(d_in, want, RTOL_ACT, "rounded conv_bwd_input")
    assert np.abs(host(binding.conv_bwd_input(dev(d), dev(k), H, W)) - want).max() > 20 * np.abs(d_in - want).max()


# besides: channel counts on both sides of eight and a last group of eight images with one, seven and eight of them
@pytest.mark.parametrize("case", CASES + [(7, 8, 10, 10, 8, 3, 3), (8, 9, 10, 10, 17, 3, 3), (257, 7, 12, 12, 33, 5, 5)])
def test_tiled_convolutions_bf16(case):
    B, Cin, H, W, Cout, KH, KW = case
    x = oracle.round_bf16(inputs.make_signed((B, Cin, H, W), 81))
    k = oracle.round_bf16(inputs.make_signed((Cout, Cin, KH, KW), 82))
    d = oracle.round_bf16(inputs.make_signed((B, Cout, H - KH + 1, W - KW + 1), 83))
    p_k, p_b = weight_gradient(x, d, KH, KW)
    x, k, d, b = dev(x), dev(k), dev(d), dev(inputs.make_signed((Cout,), 84))  # rounding again changes nothing
    assert_close(host(binding.conv_fwd(x, k, b, bf16=True)), host(binding.conv_fwd(x, k, b, valu=True)).astype(np.float64),
                 RTOL_ACT, "tiled conv_fwd_bf16")
    assert_close(host(binding.conv_bwd_input(d, k, H, W, bf16=True)),
                 host(binding.conv_bwd_input(d, k, H, W, valu=True)).astype(np.float64), RTOL_ACT, "tiled conv_bwd_input_bf16")
    d_k, d_b = binding.conv_bwd_weight(x, d, bf16=True)
    assert_close(host(d_k), p_k, RTOL_ACT, "tiled conv_bwd_weight_bf16")
    assert_close(host(d_b), p_b, RTOL_ACT, "tiled conv_bwd_bias_bf16")
    again, none = binding.conv_bwd_weight(x, d, want_bias=False, bf16=True)
    assert none is None and torch.equal(again, d_k)


@pytest.mark.parametrize("B,I,O", [(300, 784, 100), (17, 4096, 40), (1000, 64, 16), (33, 250, 250), (1, 192, 11)])
def test_tiled_fully_connected(B, I, O):
    x, w, b = inputs.make_signed((B, I), 75), inputs.make_signed((O, I), 76), inputs.make_signed((O,), 77)
    d = inputs.make_signed((B, O), 78)
    x64, w64, d64 = x.astype(np.float64), w.astype(np.float64), d.astype(np.float64)
    assert_close(host(binding.fc_fwd(dev(x), dev(w), dev(b))), x64 @ w64.T + b, RTOL_ACT, "tiled fc_fwd")
    assert_close(host(binding.fc_bwd_input(dev(d), dev(w))), d64 @ w64, RTOL_ACT, "tiled fc_bwd_input")
    d_w, d_b = binding.fc_bwd_weight(dev(x), dev(d))
    assert_close(host(d_w), d64.T @ x64, RTOL_ACT, "tiled fc_bwd_weight")
    assert_close(host(d_b), d64.sum(axis=0), RTOL_ACT, "tiled fc_bwd_bias")
