"""Which kernels of the factorisation the sizes of test_gpu_factor.py reach, from the work lists' formulas: a cluster of nt tiles of 64
has ceil(nt / 2) block columns; step k multiplies the blocks below block column k; a tree level of children of `half` tiles takes
half / 2 times the block rows of every second child."""
import os
import re

from test_gpu_factor import SIZES

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_12128_amd", "csrc", "factor.hip")


def shared_by(items, k):
    """How many workgroups share a block's sum in step k: the number that fills the last round of two workgroups on each of 256
    compute units best."""
    cost = {}
    for p in range(1, 9):
        if p == 1 or 2 * p <= k:
            rounds, left = divmod(items * p, 512)
            cost[p] = (2.0 * rounds + (0.0, 1.6, 2.0)[-(-left // 256)]) * (8.0 * k / p + 45.0)
    return min(cost, key=lambda p: (cost[p], p))


def launches(sizes):
    nt = [-(-b // 64) for b in sizes]
    nb = [(t + 1) // 2 for t in nt]
    steps = [(k, sum(max(0, x - k - 1) for x in nb)) for k in range(max(nb))]
    tree, half = [], 2
    while half < max(nt):
        tree.append(sum(half // 2 * min(half // 2, (t - mid + 1) // 2) for t in nt for mid in range(half, t, 2 * half)))
        half *= 2
    return steps, tree


def test_every_route_of_the_factorisation_is_tested():
    few = int(re.search(r"constexpr uint64_t FEW_BLOCKS = (\d+);", open(SOURCE).read()).group(1))
    multiply, tree, shared = set(), set(), set()
    for sizes in SIZES.values():
        steps, levels = launches(sizes)
        ragged = any(-(-b // 64) % 2 for b in sizes)          # a block with one row tile
        for k, items in steps:
            if items:
                multiply.add((items > few, ragged))
                shared.add((items > few, shared_by(items, k) > 1))
        tree |= {(items > few, ragged) for items in levels}
    for routes in (multiply, tree):
        assert {(False, True), (True, True)} <= routes
    assert {(False, False), (False, True), (True, False), (True, True)} <= shared
