"""The network in 64 bits, its linear parts optionally as sums of products of bfloat16 pieces, and an estimate of which of those
products a result lacks.

An operand of the pieces is x = h + m + l, each piece the bfloat16 nearest to what is left.  The products that a result has to
hold are all but m l, l m and l l, which together are below 2^-24 of the whole; each of the others, left out, moves the result
in a direction of its own, known in 64 bits.  `missing` fits a result's distance from the exact one by those directions: 1 for a
product that is left out, 0 for one that is there.  Rounding has no part in any of the directions, so thousands of results show
a product far below the error of a single one."""
import numpy as np
import torch
import torch.nn.functional as F

SMALL_PRODUCTS = ((0, 1), (1, 0), (1, 1), (0, 2), (2, 0))  # pieces of the first and the second operand
LOG2E = float(np.float32(np.log2(np.e)))


def pieces(x):
    """Three tensors of 64-bit floats that hold bfloat16 values, from one that holds fp32 values."""
    out, rest = [], x.float()
    for _ in range(3):
        p = rest.to(torch.bfloat16).float()
        out.append(p.double())
        rest = rest - p
    return out


def missing(got, want, without):
    """Share of each product that `got` lacks: got - want fitted by without[i] - want."""
    a = np.stack([np.asarray(x - want, np.float64).ravel() for x in without], axis=1)
    norm = np.linalg.norm(a, axis=0)
    fit = np.linalg.lstsq(a / norm, np.asarray(got, np.float64).ravel() - np.asarray(want).ravel(), rcond=None)[0]
    return fit / norm


def forward(x, k, b):
    """Convolution, bias and sigmoid."""
    return torch.sigmoid(F.conv2d(x, k, b))


def layer(x, k, b, scale, pooled=1.0):
    """Convolution layer of fp32 operands and, per small product, the layer without it.  The kernel cuts x / pooled, which is
    exact, and the weights times the fp32 number pooled * scale."""
    x, k = x / pooled, k * np.float32(pooled * scale)
    z = F.conv2d(x.double(), k.double()) / scale + b.double().view(1, -1, 1, 1)
    px, pk = pieces(x), pieces(k)
    return torch.sigmoid(z), [torch.sigmoid(z - F.conv2d(px[i], pk[j]) / scale) for i, j in SMALL_PRODUCTS]


def weight_gradient(x, d):
    """Sum over images and pixels of d[j] times the patches of x, for every small product the sum without it too."""
    g = lambda a, e: F.conv2d(a.transpose(0, 1), e.transpose(0, 1)).transpose(0, 1)
    px, pd = pieces(x), pieces(d)
    want = g(x.double(), d.double())
    return want, [want - g(px[j], pd[i]) for i, j in SMALL_PRODUCTS]


def input_gradient(d, k):
    """The layer's input error, for every small product without it too."""
    pd, pk = pieces(d), pieces(k)
    want = F.conv_transpose2d(d.double(), k.double())
    return want, [want - F.conv_transpose2d(pd[i], pk[j]) for i, j in SMALL_PRODUCTS]


def up(d):
    """backavgpool."""
    return 0.25 * d.repeat_interleave(2, 2).repeat_interleave(2, 3)


def gradients(w, images, labels):
    """Gradients of both convolution layers' weights summed over the images, in 64 bits, each with its versions without one small
    product: of the second layer's weight gradient, and of its input error for the first layer's."""
    t = {n: torch.from_numpy(np.asarray(v, np.float64)) for n, v in w.items()}
    k1, k2, fc = t["k1"].view(6, 1, 5, 5), t["k2"].view(12, 6, 5, 5), t["fc"].view(10, 192)
    x = torch.from_numpy(images.astype(np.float64)).view(-1, 1, 28, 28)
    c1 = forward(x, k1, t["b1"])
    s1 = F.avg_pool2d(c1, 2)
    c2 = forward(s1, k2, t["b2"])
    s2 = F.avg_pool2d(c2, 2)
    y = torch.sigmoid(s2.view(-1, 192) @ fc.T + t["b"])
    delta = (y - F.one_hot(torch.from_numpy(labels).long(), 10)) * y * (1 - y)
    d_c2 = up((delta @ fc).view(-1, 12, 4, 4)) * c2 * (1 - c2)
    as_fp32 = lambda a: a.float().double()
    g_k2 = weight_gradient(as_fp32(4.0 * s1), as_fp32(d_c2))
    d_s1, less = input_gradient(as_fp32(d_c2), k2)
    first = lambda d: weight_gradient_64(x, up(d) * c1 * (1 - c1))
    return ((0.25 * g_k2[0]).numpy(), [(0.25 * g).numpy() for g in g_k2[1]]), (first(d_s1).numpy(), [first(d).numpy() for d in less])


def weight_gradient_64(x, d):
    return F.conv2d(x.transpose(0, 1), d.transpose(0, 1)).transpose(0, 1)
