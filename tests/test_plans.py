"""Launch plans, seen through the size queries of the weight gradients (host-only logic: no GPU needed)."""
import concurrent.futures
import random
import statistics
import time

from paper_1912_05234_amd import binding


def layers(n, seed):
    """Layers of the kind and the sizes that the performance cases draw, hardly ever one twice."""
    rng = random.Random(seed)
    out = []
    for _ in range(n):
        k = rng.choice([1, 2, 3, 4, 5, 7])
        out.append((rng.randint(1, 4000), rng.randint(1, 32), rng.randint(k + 1, 40), rng.randint(k + 1, 40), rng.randint(1, 32), k, k))
    return out


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


def test_layers_of_one_unit_per_workgroup_take_no_five_tap_tiles():
    """Columns of partial sums, which is what these layers ask for: with five tap tiles they were 48, 36 and 52, and such calls
    up to a fifth slower."""
    L = binding.lib()
    for shape, columns in (((16, 24, 30, 37, 17, 7, 7), 30), ((12, 16, 28, 36, 27, 7, 7), 20), ((13, 16, 36, 37, 14, 5, 5), 39)):
        B, Cin, H, W, Cout, KH, KW = shape
        assert L.cnn_conv_bwd_weight_workspace_bytes(*shape) == columns * 4 * (Cout * Cin * KH * KW + Cout)


def test_plans_do_not_depend_on_what_was_planned_before():
    """More layers than the table of plans holds, from eight threads, each in an order of its own."""
    L = binding.lib()
    shapes = layers(700, 5)

    def ask(seed):
        order = list(range(len(shapes)))
        random.Random(seed).shuffle(order)
        got = {}
        for i in order + order[:100]:
            both = L.cnn_conv_bwd_weight_workspace_bytes(*shapes[i]), L.cnn_conv_bwd_weight_bf16_workspace_bytes(*shapes[i])
            assert got.setdefault(i, both) == both
        return got

    alone = ask(0)
    with concurrent.futures.ThreadPoolExecutor(8) as pool:
        assert all(got == alone for got in pool.map(ask, range(1, 9)))


def test_planning_a_new_layer_is_cheap():
    """A program whose batch or image size changes from call to call plans every time: 4 us of host time in the median
    for a weight gradient, so that the query takes five to six times what that of a known layer takes through ctypes (17 to
    20 times with every candidate evaluated).  The best of several sets, for a busy machine."""
    L = binding.lib()

    def median(shapes):
        times = []
        for shape in shapes:
            t = time.perf_counter()
            L.cnn_conv_bwd_weight_workspace_bytes(*shape)
            times.append(time.perf_counter() - t)
        return statistics.median(times)

    known = layers(1, 9) * 1000
    ratios = [median(layers(1000, seed)) / median(known) for seed in (6, 7, 8, 10)]
    assert min(ratios) < 12, ratios


def test_a_loop_over_forty_batch_sizes_plans_each_once():
    L = binding.lib()
    shapes = [(batch, 9, 31, 29, 21, 3, 3) for batch in range(100, 140)]

    def once():
        t = time.perf_counter()
        for shape in shapes:
            L.cnn_conv_bwd_weight_workspace_bytes(*shape)
        return time.perf_counter() - t

    first = once()
    assert min(once() for _ in range(5)) < first / 2
